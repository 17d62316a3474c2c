"""The tile autotuner times the run lengths that it records, on the CPU: the batched
launches over its object take every candidate as it is, and the table shipped with
the package belongs to the library that is built."""
from __future__ import annotations

import json

import pytest

from paper_2503_01582_amd import api, autotune
from plan_driver import run_plan_program


@pytest.mark.parametrize("n_rays", [autotune.N_RAYS, 16384, 3 * 4096])
def test_candidates_run_as_asked(tmp_path, n_rays):
    fwd = autotune.candidates(n_rays, autotune.FWD_CANDIDATES)
    bwd = autotune.candidates(n_rays, autotune.BWD_CANDIDATES)
    if n_rays == autotune.N_RAYS:
        assert tuple(fwd) == autotune.FWD_CANDIDATES and tuple(bwd) == autotune.BWD_CANDIDATES
    out = run_plan_program(tmp_path, f"""
    const std::vector<int64_t> tiles(1, {n_rays * autotune.SAMPLES // 16});
    for (int64_t c : {{{", ".join(map(str, fwd))}}}) {{
        const int64_t run = host::run_length(tiles, c, host::kFwdQuantum, kCus);
        CHECK(run == c, "forward: asked for %d, runs %d\\n", (int)c, (int)run);
    }}
    for (int width : {{32, 64, 128}})
        for (int64_t c : {{{", ".join(map(str, bwd))}}}) {{
            const MlpShape m{{16, width, 1, PRENOM_BF16}};
            const int64_t run = host::run_length(tiles, c, host::kBwdQuantum, kCus * host::bwd_blocks_per_cu(m));
            CHECK(run == c, "backward: asked for %d, runs %d\\n", (int)c, (int)run);
        }}
""", headers=("mlp_runs.h",))
    assert out == "ok\n", out


def test_too_few_rays_are_refused():
    with pytest.raises(ValueError):
        autotune.candidates(1000, autotune.FWD_CANDIDATES)


def test_packaged_table_is_of_this_library():
    with open(autotune.PACKAGED) as f:
        keys = list(json.load(f))
    assert keys and all(k.split("|")[2] == api.version() for k in keys)
