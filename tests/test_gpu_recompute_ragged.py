"""The recompute form whose last pass is shorter than the others, at sizes whose
passes split the table tiles differently: its table gradient against the stored
form's on the same samples.  A pass rounds its fixed-point sums to FP32 and adds
them, so a row carries one rounding of each pass's sum and one of each addition:
with two or three passes at most six of 2^-24, of values about as large as the
largest gradient.  The last shape's stored form has tiles of one range of 8751
blocks, more than a workgroup keeps the segment bounds of."""
from __future__ import annotations

import numpy as np
import pytest

from parity_util import rel_errors
from synth.arch import Arch
from synth.params import init_params
from synth.workloads import SampleSpec, small_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("levels,log2t,S,rays", [(16, 18, 56, 70001), (8, 10, 40, 62326), (16, 17, 63, 66280), (8, 20, 64, 70001)])
def test_ragged_last_pass(levels, log2t, S, rays):
    from paper_2503_01582_amd import api
    print(f"test_ragged_last_pass: {levels} levels of 2^{log2t}, {rays} rays x {S}", flush=True)
    arch = Arch(n_levels=levels, log2_table=log2t, width=32, hidden=1)
    rng = np.random.default_rng([levels, log2t, S])
    b = small_batch(0, res=96)
    pick = rng.integers(0, b.rays_o.shape[0], rays)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    spec = SampleSpec(n_coarse=0, n_fine=S, include_coarse=False, uniform_only=True)
    xi = rng.random((rays, S), dtype=np.float32)
    samp = api.prenom_sample(spec, dev(b.rays_o[pick]), dev(b.rays_d[pick]), dev(xi), b.world_to_obj)
    params = init_params(arch, 3)
    params[:arch.n_table_params] *= 1e3
    model = api.Model(arch, params)
    d_rgb = dev(rng.normal(size=(rays, 3)).astype(np.float32))
    got = []
    for recompute in (False, True):
        ws = torch.empty(api.prenom_workspace_size(arch, rays, S, recompute=recompute), dtype=torch.uint8, device="cuda")
        model.grads.zero_()
        api.prenom_render_fwd(model, samp, None, ws, want_loss=False, recompute=recompute)
        api.prenom_render_bwd(model, samp, None, ws, d_rgb=d_rgb, recompute=recompute)
        got.append(model.grads.cpu().numpy()[:arch.n_table_params])
        del ws
    e_max, e_2 = rel_errors(got[1], got[0])
    print(f"  max-rel {e_max:.2e}, 2-rel {e_2:.2e}", flush=True)
    assert np.abs(got[0]).max() > 0 and e_max <= 2.0 ** -21 and e_2 <= 2.0 ** -21
