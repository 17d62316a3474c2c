"""The 128-wide FP32 weight gradient of a batch: few ranges give each range's
rows and columns to four blocks, many give a range to one.  The same sums cut
into 3 and into 70 ranges, against each other: FP32 sums of 35840 terms in
another order, so each within sqrt(35840) 2^-24 of the terms' size, and the
whole gradient within 1e-5 of its norm."""
from __future__ import annotations

import numpy as np
import pytest

from synth.workloads import LossSpec
from test_gpu_encode_lds import params_of, samples

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,D", [(8, 1), (12, 2), (16, 2)])
def test_ranges_of_the_wide_weight_gradient(L, D):
    print(f"test_ranges_of_the_wide_weight_gradient[{L}, {D}]", flush=True)
    from paper_2503_01582_amd import batch as B
    from synth.arch import Arch
    n, S = 560, 64
    arch = Arch(n_levels=L, log2_table=14, width=128, hidden=D)
    samp = samples(n, S, 5)
    g = torch.Generator().manual_seed(1)
    kw = dict(tgt_rgb=torch.rand((n, 3), generator=g).cuda(), tgt_depth=torch.rand(n, generator=g).cuda(),
              mask=torch.ones(n, dtype=torch.uint8, device="cuda"))
    grads = []
    for bwd_tiles in (1024, 32):
        tiles = [dict(in_dim=2 * L, width=128, hidden=D, dtype="fp32", fwd_tiles=64, bwd_tiles=bwd_tiles)]
        bm = B.BatchModel([B.BatchObject(arch, n, None, np.eye(3, 4, dtype=np.float32))], [params_of(arch, 3)],
                          tiles=tiles)
        ws = B.alloc_workspace(bm, S)
        loss = LossSpec(0, 0.0, 0.0)
        B.prenom_batch_render_fwd(bm, samp, loss, ws, **kw)
        bm.grads.zero_()
        B.prenom_batch_render_bwd(bm, samp, loss, ws, **kw)
        torch.cuda.synchronize()
        grads.append(bm.object_grads(0)[arch.n_table_params:].double().cpu())
    a, b = grads
    assert float(a.norm()) > 0
    assert float((a - b).norm()) <= 1e-5 * float(a.norm())
