"""The hash-table gradient at the edges of its item sizes: sample counts around
one 512-sample block, rays without a gradient inside a block, levels of one
table tile and of many, tables whose tiles are reduced in one range of blocks
and in several, and both record formats, against the FP64 oracle; and the
gradient's bits from one run to the next."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as orc
from parity_util import TOL_FP32, assert_close, relu_stable_rays
from synth.arch import Arch
from synth.params import init_params
from synth.workloads import SampleSpec, small_batch, uniform_xi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# Compact records keep each contribution within 2^-15 of its larger feature;
# an entry whose contributions cancel down to an eighth of their absolute sum
# is then off by 2^-12 of itself.
TOL_COMPACT = 2.0 ** -12

# (levels, log2 table, rays, samples per ray, table type)
SHAPES = [(8, 10, 1, 3, "fp32"),       # fewer samples than a wave, every level one tile
          (8, 14, 73, 7, "fp32"),      # 511 samples
          (12, 17, 57, 9, "fp32"),     # 513
          (8, 19, 256, 4, "fp32"),     # two whole blocks, 64 tiles
          (16, 15, 2049, 31, "fp32"),  # a ragged last block; tiles in one range
          (8, 14, 4099, 33, "fp32"),   # tiles in several ranges
          (8, 21, 300, 17, "fp32"),    # 256 tiles a level
          (8, 14, 4099, 33, "fp16"),
          (12, 18, 301, 17, "fp16")]


@pytest.mark.parametrize("levels,log2t,rays,S,table", SHAPES)
def test_table_gradient_edges(levels, log2t, rays, S, table):
    from paper_2503_01582_amd import api
    print(f"test_table_gradient_edges: {levels} levels of 2^{log2t}, {rays} rays x {S}, {table} table", flush=True)
    arch = Arch(n_levels=levels, log2_table=log2t, width=32, hidden=1, table_dtype=table)
    rng = np.random.default_rng([levels, log2t, rays, S])
    b = small_batch(0, res=96)
    pick = rng.integers(0, b.rays_o.shape[0], rays)
    b.rays_o, b.rays_d, b.xi = b.rays_o[pick], b.rays_d[pick], uniform_xi(rng, rays, S)
    spec = SampleSpec(n_coarse=0, n_fine=S, include_coarse=False, uniform_only=True)
    o = orc.sample(b.rays_o, b.rays_d, b.xi, n_coarse=0, n_fine=S, include_coarse=False, uniform_only=True,
                   eps=spec.eps, near=spec.near, far=spec.far, world_to_obj=b.world_to_obj)
    geo = (o["ray_obj"].astype(np.float32), o["t"].astype(np.float32), o["dt"].astype(np.float32), o["flags"])
    params = init_params(arch, 3)
    params[:arch.n_table_params] *= 1e3
    emulate = table == "fp16"
    d_rgb = rng.normal(size=(rays, 3)).astype(np.float32)
    d_rgb[rng.random(rays) < 0.3] = 0.0  # rays without a gradient among the others
    d_rgb[~relu_stable_rays(arch, params, geo, rng, emulate=emulate, rel=1e-6)] = 0.0
    ref = orc.render_bwd(arch, params, *geo, d_rgb=d_rgb, emulate=emulate)

    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    model = api.Model(arch, params)
    samp = api.SampleOut(ray_obj=dev(geo[0]), t=dev(geo[1]), dt=dev(geo[2]), bins=None, flags=dev(geo[3]))
    ws = api.Workspace().get(arch, rays, S)
    api.prenom_render_fwd(model, samp, None, ws, want_loss=False)
    got = []
    for _ in range(2):
        model.grads.zero_()
        api.prenom_render_bwd(model, samp, None, ws, d_rgb=dev(d_rgb))
        got.append(model.grads.cpu().numpy()[:arch.n_table_params])
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32)), "the gradient's bits depend on the run"
    assert_close(got[0], ref[:arch.n_table_params], tol=TOL_COMPACT if emulate else TOL_FP32, name="table gradient")
