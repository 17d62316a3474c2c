"""The canonical yaw search's workspace on the CPU: it holds the split of every
call, and a workspace of the largest cloud and most yaws does for smaller ones."""
from __future__ import annotations

from plan_driver import run_plan_program

SWEEP = r"""
    std::vector<int64_t> points;
    for (int64_t n = 1; n < 20000; n += 1 + n / 64) points.push_back(n);
    for (int64_t n = 20000; n <= PRENOM_MAX_YAW_POINTS && n < 400000000; n += n / 41) points.push_back(n);
    for (int64_t n : {2048, 2049, 65536, 65537, 1 << 20, (1 << 20) + 1, 8927, 60000}) points.push_back(n);
    for (int K = 1; K <= PRENOM_MAX_YAWS; K += K < 800 ? 1 : 97)
        for (int64_t n : points) {
            YawArgs a{};
            a.n = n;
            a.K = K;
            yaw_split(a);
            CHECK(yaw_doubles(a) <= yaw_doubles_most(n, K), "%lld points x %d: %zu > %zu\n", (long long)n, K,
                  yaw_doubles(a), yaw_doubles_most(n, K));
        }
"""


def test_workspace_holds_every_split(tmp_path):
    out = run_plan_program(tmp_path, SWEEP)
    assert out == "ok\n", out


def test_workspace_size_grows():
    from paper_2503_01582_amd import _lib
    size = _lib.lib().prenom_canonical_yaw_workspace_size
    points = sorted({*range(1, 3000, 13), *range(3000, 80000, 997), 65536, 65537, 1 << 20, (1 << 20) + 1})
    yaws = sorted({*range(1, 400, 3), 64, 65, 360, 720, 1000})
    last = {}
    for n in points:
        before = 0
        for k in yaws:
            need = size(n, k)
            assert need >= before and need >= last.get(k, 0), f"{n} points x {k} yaws need {need} bytes"
            before = last[k] = need
