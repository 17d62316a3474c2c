"""The plan of the hash-table gradient's scatter against the workspace that is
reserved for it, on the CPU: a pass over fewer samples than the workspace was
laid out for (the last pass of the recompute form) has to fit every array of
the longest one, and a workspace of the largest call has to do for the smaller
ones."""
from __future__ import annotations

import pytest

from plan_driver import run_plan_program
from synth.arch import Arch

SWEEP = r"""
    for (int L = 1; L <= PRENOM_MAX_LEVELS; ++L)
        for (int log2T = 10; log2T <= 24; log2T += L % 4 == 0 ? 1 : 3) {
            GridInfo g{};
            g.n_levels = L;
            g.log2_table = log2T;
            for (int l = 0; l < L; ++l) {  // 16 to 2048, geometric
                double r = 16.0;
                for (int k = 0; k < l; ++k) r *= 1.3819;
                g.res[l] = (int)r;
                const int64_t side = g.res[l] + 1;
                if (side * side * side <= (int64_t)1 << log2T) g.dense_mask |= 1u << l;
            }
            // every length of a pass in blocks of 512 samples, up to 2^21 samples and a block more
            ScatterObj p = scatter_plan(g, 1);
            for (int64_t nb = 2; nb <= 4097; ++nb) {
                const ScatterObj o = scatter_plan(g, 512 * nb);
                CHECK(o.n_parts >= p.n_parts && o.n_ritems >= p.n_ritems && o.n_ctiles >= p.n_ctiles,
                      "%d levels of 2^%d: %lld blocks need %d parts, %lld need %d\n", L, log2T, (long long)nb,
                      (int)o.n_parts, (long long)nb - 1, (int)p.n_parts);
                CHECK(scatter_items(o) > scatter_items(p) && scatter_records(o) > scatter_records(p) &&
                          scatter_segs(o) > scatter_segs(p),
                      "%d levels of 2^%d: arrays of %lld blocks\n", L, log2T, (long long)nb);
                for (int l = 0; l < L; ++l) CHECK(o.split[l] >= 1 && o.split[l] <= nb, "split\n");
                p = o;
            }
        }
"""


def test_shorter_passes_fit_the_longest(tmp_path):
    out = run_plan_program(tmp_path, SWEEP)
    assert out == "ok\n", out


@pytest.mark.parametrize("recompute", [False, True])
@pytest.mark.parametrize("levels,log2t,S", [(16, 18, 56), (8, 10, 40), (16, 17, 63), (12, 15, 64), (16, 19, 64)])
def test_workspace_size_grows_with_the_rays(levels, log2t, S, recompute):
    from paper_2503_01582_amd import api
    arch = Arch(n_levels=levels, log2_table=log2t, width=32, hidden=1)
    last = 0
    for blocks in range(1, 6000, 1):
        n = blocks * 512 // S
        size = api.prenom_workspace_size(arch, n, S, recompute=recompute)
        assert size >= last, f"{n} rays need {size} bytes, fewer rays {last}"
        last = size
