"""The hash-table gradient far from one: an upstream gradient scaled by a power
of two scales the table gradient by it, from feature gradients near the smallest
normal number to ones near the largest, in both record formats and in whole and
split tiles; and samples whose gradient is not finite leave the others'
contributions as they are."""
from __future__ import annotations

import numpy as np
import pytest

from parity_util import rel_errors
from synth.arch import Arch
from synth.params import init_params
from synth.workloads import SampleSpec, small_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def case(levels, log2t, rays, S, table="fp32", up=0):
    """Architecture, random upstream gradients and the table gradient of a
    uniform-sampling render; the feature gradients are 2^up times larger (the
    first layer's weights are, and the features as much smaller)."""
    from paper_2503_01582_amd import api
    arch = Arch(n_levels=levels, log2_table=log2t, width=32, hidden=1, table_dtype=table)
    rng = np.random.default_rng([levels, log2t, rays, S])
    b = small_batch(0, res=96)
    pick = rng.integers(0, b.rays_o.shape[0], rays)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    spec = SampleSpec(n_coarse=0, n_fine=S, include_coarse=False, uniform_only=True)
    samp = api.prenom_sample(spec, dev(b.rays_o[pick]), dev(b.rays_d[pick]), dev(rng.random((rays, S), dtype=np.float32)),
                             b.world_to_obj)
    params = init_params(arch, 3)
    params[:arch.n_table_params] *= 1e3 * 2.0 ** -up
    params[arch.n_table_params:arch.n_table_params + arch.width * arch.in_dim] *= 2.0 ** up
    model = api.Model(arch, params)
    ws = api.Workspace().get(arch, rays, S)
    api.prenom_render_fwd(model, samp, None, ws, want_loss=False)

    def table_gradient(d_rgb):
        model.grads.zero_()
        api.prenom_render_bwd(model, samp, None, ws, d_rgb=dev(d_rgb))
        return model.grads.cpu().numpy()[:arch.n_table_params]

    return arch, rng.normal(size=(rays, 3)).astype(np.float32), table_gradient


# The MLP's products and the contributions are FP32 down to 2^-149.  With the
# largest row about 2^-110, the absolute roundings of subnormal numbers (2^-150
# each, some 2^13 of them in a row) are 2^-27 of it.
@pytest.mark.parametrize("levels,log2t,rays,S,table", [(8, 14, 511, 9, "fp32"), (8, 11, 4099, 33, "fp32"),
                                                       (12, 17, 301, 17, "fp16")])
@pytest.mark.parametrize("target", [-30, -60, -100, -110])
def test_scaled_gradient(levels, log2t, rays, S, table, target):
    print(f"test_scaled_gradient: {levels} levels of 2^{log2t}, {rays} rays x {S}, {table}, 2^{target}", flush=True)
    arch, d_rgb, table_gradient = case(levels, log2t, rays, S, table)
    ref = table_gradient(d_rgb)
    shift = target - int(np.floor(np.log2(np.abs(ref).max())))
    got = table_gradient(np.ldexp(d_rgb, shift))
    e_max, e_2 = rel_errors(np.ldexp(got.astype(np.float64), -shift), ref)
    print(f"  shift {shift}: max-rel {e_max:.2e}, 2-rel {e_2:.2e}", flush=True)
    assert e_max <= 2.0 ** -20 and e_2 <= 2.0 ** -20


# Above 2^124 a wave's runs are not merged, so the records are others: each keeps
# its larger feature to 2^-22 in nearest rounding, as the merged ones do.
def test_large_gradient():
    print("test_large_gradient", flush=True)
    arch, d_rgb, table_gradient = case(8, 14, 511, 9, up=12)
    ref = table_gradient(d_rgb)
    shift = 126 - int(np.floor(np.log2(np.abs(ref).max())))
    got = table_gradient(np.ldexp(d_rgb, shift))
    e_max, e_2 = rel_errors(np.ldexp(got.astype(np.float64), -shift), ref)
    print(f"  shift {shift}: max-rel {e_max:.2e}, 2-rel {e_2:.2e}", flush=True)
    assert e_max <= 2.0 ** -20 and e_2 <= 2.0 ** -20


@pytest.mark.parametrize("levels,log2t,rays,S,table", [(8, 14, 511, 9, "fp32"), (8, 11, 4099, 33, "fp32"),
                                                       (12, 17, 301, 17, "fp16")])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_samples_leave_the_others(levels, log2t, rays, S, table, value):
    """The bits of the gradient with those rays' upstream gradient zero."""
    print(f"test_non_finite_samples_leave_the_others: {levels} levels of 2^{log2t}, {rays} rays x {S}, {table}, {value}",
          flush=True)
    arch, d_rgb, table_gradient = case(levels, log2t, rays, S, table)
    bad = np.arange(5, rays, 37)
    d_rgb[bad] = 0.0
    ref = table_gradient(d_rgb)
    d_rgb[bad, bad % 3] = value
    got = table_gradient(d_rgb)
    assert np.abs(ref).max() > 0 and np.array_equal(got.view(np.uint32), ref.view(np.uint32))


# 2^22 samples over levels of 2^24 rows, a tenth of the rays 2^-20 of the others.
# With M the largest feature gradient, a tile of a hashed level gets at most two
# records of a block on average, so its sums stay below 2 * 8 M * 8192 = 2^17 M and
# its scale is at least 2^44 / M (coarser ones, of the level's 2^22 M, 2^39 / M): a
# record is rounded with an RMS error of 2^-45 M / sqrt(3), and a row that only the
# small rays reach holds a few.  M is taken as the large rays' largest row of the
# finest level, whose rows hold a few samples as well.
def test_small_rows_of_large_tables():
    from paper_2503_01582_amd import api
    print("test_small_rows_of_large_tables", flush=True)
    rays, S = 65536, 64
    arch = Arch(n_levels=8, log2_table=24, width=32, hidden=1, resolutions=(16, 32, 64, 128, 256, 512, 1024, 2048))
    gen = torch.Generator("cuda").manual_seed(3)
    rand = lambda *shape: torch.rand(shape, device="cuda", generator=gen)
    o = torch.randn((rays, 3), device="cuda", generator=gen)
    o = 1.5 * o / o.norm(dim=1, keepdim=True)
    d = rand(rays, 3) * 0.9 - 0.45 - o
    d = d / d.norm(dim=1, keepdim=True)
    spec = SampleSpec(n_coarse=0, n_fine=S, include_coarse=False, uniform_only=True)
    samp = api.prenom_sample(spec, o, d, rand(rays, S), small_batch(0).world_to_obj)
    params = init_params(Arch(n_levels=8, log2_table=10, width=32, hidden=1), 3)[-arch.n_mlp_params:]
    model = api.Model(arch, np.zeros(arch.n_params, np.float32))
    model.params[arch.n_table_params:] = torch.as_tensor(params).cuda()
    model.params[:arch.n_table_params] = rand(arch.n_table_params) * 0.2 - 0.1
    ws = api.Workspace().get(arch, rays, S)
    api.prenom_render_fwd(model, samp, None, ws, want_loss=False)
    d_rgb = torch.randn((rays, 3), device="cuda", generator=gen)
    small = (rand(rays) < 0.1)[:, None]

    def table_gradient(up):
        model.grads.zero_()
        api.prenom_render_bwd(model, samp, None, ws, d_rgb=up.contiguous())
        return model.grads[:arch.n_table_params].clone()

    zero = torch.zeros_like(d_rgb)
    large = table_gradient(torch.where(small, zero, d_rgb))
    ref = table_gradient(torch.where(small, d_rgb * 2.0 ** -20, zero))
    got = table_gradient(torch.where(small, d_rgb * 2.0 ** -20, d_rgb))
    rows = (large == 0) & (ref != 0)
    M = float(large[-2 << arch.log2_table:].abs().max())
    rms = float((got[rows].double() - ref[rows].double()).square().mean().sqrt())
    print(f"  {int(rows.sum())} rows, rms 2^{np.log2(rms / M):.1f} M, rows' own rms "
          f"2^{np.log2(float(ref[rows].double().square().mean().sqrt()) / M):.1f} M", flush=True)
    assert int(rows.sum()) > 100000 and rms <= 2.0 ** -43 * M
