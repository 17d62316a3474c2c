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


MIXED = r"""
    srand(5);
    for (int trial = 0; trial < 4000; ++trial) {
        std::vector<ScatterObj> objs(1 + rand() % 48);
        int64_t records = 0;
        for (ScatterObj& o : objs) {
            GridInfo g{};
            g.n_levels = 1 + rand() % PRENOM_MAX_LEVELS;
            g.log2_table = 10 + rand() % 15;
            for (int l = 0; l < g.n_levels; ++l) {
                g.res[l] = 2 + rand() % 400;
                const int64_t side = g.res[l] + 1;
                if (side * side * side <= (int64_t)1 << g.log2_table) g.dense_mask |= 1u << l;
            }
            o = scatter_obj(g, (int64_t)(rand() % 1000) << rand() % 15);
            records += scatter_records(o);
        }
        int64_t parts = 0;
        for (ScatterObj& o : objs) {
            scatter_split(o, records);
            parts += o.n_parts;
        }
        CHECK(parts <= scatter_parts_most(records), "trial %d: %lld records need %lld parts, reserved %lld\n", trial,
              (long long)records, (long long)parts, (long long)scatter_parts_most(records));
    }
    for (int64_t r = 0; r < 40000000; r += 4096)
        CHECK(scatter_parts_most(r) <= scatter_parts_most(r + 4096), "%lld records\n", (long long)r);
"""


def test_parts_of_a_batch_pass_fit(tmp_path):
    out = run_plan_program(tmp_path, MIXED)
    assert out == "ok\n", out


def batch_size(shapes, rays, S, tiles=()):
    """Workspace of a batch of objects, from its sizes alone."""
    import ctypes as C

    from paper_2503_01582_amd import _lib as L
    from paper_2503_01582_amd import batch as B
    from synth.workloads import nocs_affine
    objs = B._c_objects([B.BatchObject(a, n, None, nocs_affine()) for a, n in zip(shapes, rays)])
    b = L.PrenomBatch()
    b.n_objects, b.objects = len(shapes), C.cast(objs, C.POINTER(L.PrenomObject))
    arr, b.n_tiles = B._c_tiles(tiles)
    b.tiles = C.cast(arr, C.POINTER(L.PrenomMlpTiles))
    size = L.lib().prenom_batch_workspace_size(C.byref(b), S)
    assert size > 0
    return size


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("width", [32, 128])
def test_batch_workspace_size_grows_with_an_object(width, dtype):
    """One of three objects grows from nothing through the lengths at which the
    MLP runs and the scatter's ranges change; the batch stays one scatter pass."""
    shapes = [Arch(n_levels=8, log2_table=14, width=width, hidden=2, mlp_dtype=dtype),
              Arch(n_levels=16, log2_table=17, width=32, hidden=1, mlp_dtype=dtype),
              Arch(n_levels=8, log2_table=11, width=width, hidden=2, mlp_dtype=dtype)]
    S, last = 16, 0
    for n in list(range(0, 9000, 37)) + list(range(9000, 60000, 997)):
        size = batch_size(shapes, [n, 3000, 800], S)
        assert size >= last, f"{n} rays need {size} bytes, fewer rays {last}"
        last = size
