"""The encoding that stages a level's table in LDS against the one that gathers
from memory.  Both add the same products in the same order, so a forward pass
over many rays has to equal, bit for bit, the same rays in calls too small for
the staged kernel (whose agreement with the oracle other tests check)."""
from __future__ import annotations

import numpy as np
import pytest

from synth.arch import Arch
from synth.params import init_params

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SLICE = 512  # rays of a small call: 8 levels x 512 x 48 samples leave 768 a CU


def arch_of(log2T, table):
    return Arch(n_levels=8, log2_table=log2T, width=32, hidden=1, mlp_dtype="fp32" if table == "fp32" else "bf16",
                table_dtype=table)


def params_of(arch, seed):
    p = init_params(arch, seed)
    rng = np.random.default_rng(seed)
    p[:arch.n_table_params] = rng.uniform(-0.5, 0.5, arch.n_table_params).astype(np.float32)
    return p


def samples(n, S, seed):
    from paper_2503_01582_amd.api import SampleOut
    g = torch.Generator().manual_seed(seed)
    o = torch.rand((n, 3), generator=g)
    d = torch.rand((n, 3), generator=g) - 0.5
    t = torch.sort(torch.rand((n, S), generator=g), 1).values
    return SampleOut(ray_obj=torch.cat([o, d], 1).cuda(), t=t.cuda(),
                     dt=torch.full((n, S), 1.0 / S, device="cuda"),
                     bins=torch.zeros((n, 1), dtype=torch.int32, device="cuda"),
                     flags=torch.zeros(n, dtype=torch.uint8, device="cuda"))


def part(samp, a, b):
    from paper_2503_01582_amd.api import SampleOut
    return SampleOut(*(getattr(samp, k)[a:b].contiguous() for k in ("ray_obj", "t", "dt", "bins", "flags")))


def forward(model, samp):
    from paper_2503_01582_amd import api
    ws = api.Workspace().get(model.arch, samp.t.shape[0], samp.n_samples)
    out = api.prenom_render_fwd(model, samp, None, ws, want_loss=False)
    torch.cuda.synchronize()
    return [out[k] for k in ("rgb", "depth", "opacity")]


def small_calls(model, samp):
    parts = [forward(model, part(samp, a, a + SLICE)) for a in range(0, samp.t.shape[0], SLICE)]
    return [torch.cat(x) for x in zip(*parts)]


# 2^10: every level hashed or a few rows; one pass up to 128 KB, two up to 256;
# runs of a little over the shortest, and of several rounds
@pytest.mark.parametrize("log2T,table,S,rays", [(10, "fp32", 33, 1009), (14, "fp32", 33, 4001), (14, "fp32", 48, 40001),
                                                (15, "fp32", 33, 16001), (15, "fp16", 48, 2777),
                                                (16, "fp16", 33, 16001), (11, "fp16", 1, 40003)])
def test_staged_encoding_equals_gathers(log2T, table, S, rays):
    print(f"test_staged_encoding_equals_gathers[{log2T}, {table}, {S}, {rays}]", flush=True)
    from paper_2503_01582_amd import api
    arch = arch_of(log2T, table)
    model = api.Model(arch, params_of(arch, log2T), "cuda")
    samp = samples(rays, S, rays)
    for x, y in zip(forward(model, samp), small_calls(model, samp)):
        assert torch.equal(x, y)


# objects of one pass, of two and of none, with work for both and for the first alone
@pytest.mark.parametrize("table", ["fp32", "fp16"])
@pytest.mark.parametrize("counts", [(8000, 0, 9001, 700), (3001, 5, 2000, 700)])
def test_staged_batch_encoding_equals_gathers(table, counts):
    print(f"test_staged_batch_encoding_equals_gathers[{table}, {counts}]", flush=True)
    from paper_2503_01582_amd import api
    from paper_2503_01582_amd import batch as B
    logs = (14, 15, 15, 17) if table == "fp32" else (15, 16, 16, 18)
    archs = [arch_of(x, table) for x in logs]
    params = [params_of(a, 5 + i) for i, a in enumerate(archs)]
    bm = B.BatchModel([B.BatchObject(a, n, None, np.eye(3, 4, dtype=np.float32)) for a, n in zip(archs, counts)], params)
    samp = samples(sum(counts), 48, 3)
    ws = B.alloc_workspace(bm, 48)
    out = B.prenom_batch_render_fwd(bm, samp, None, ws, want_loss=False)
    torch.cuda.synchronize()
    r = 0
    for a, p, n in zip(archs, params, counts):
        if n:
            ref = small_calls(api.Model(a, p, "cuda"), part(samp, r, r + n))
            for k, y in zip(("rgb", "depth", "opacity"), ref):
                assert torch.equal(out[k][r:r + n], y)
        r += n
