"""The order in which a batched encoding deals its items to the XCDs, on the CPU:
every item once, in runs that stay on one XCD, and no XCD (a block's index modulo
8) with much more than its share of a small launch."""
from __future__ import annotations

from plan_driver import run_plan_program

ORDER = r"""
    for (int64_t n = 1; n < 70000; n += 1 + n / 50) {
        const int run_log2 = xcd_run_log2(n);
        const int64_t run = (int64_t)1 << run_log2, round = run * kXcds, grid = (n + round - 1) / round * round;
        std::vector<int> seen(n, 0), owner(n, -1);
        std::vector<int64_t> per(kXcds, 0);
        for (int64_t b = 0; b < grid; ++b) {
            const uint32_t item = xcd_item((uint32_t)b, run_log2);
            if (item >= n) continue;
            ++seen[item];
            owner[item] = (int)(b % kXcds);
            ++per[b % kXcds];
        }
        for (int64_t i = 0; i < n; ++i) {
            CHECK(seen[i] == 1, "%lld items: item %lld %d times\n", (long long)n, (long long)i, seen[i]);
            CHECK(owner[i] == owner[i - i % run], "%lld items: run of %lld split\n", (long long)n, (long long)i);
        }
        for (int64_t p : per)
            CHECK(8 * p <= n + (n < 32 ? 8 : n / 4), "%lld items: an XCD has %lld\n", (long long)n, (long long)p);
    }
"""


def test_small_launches_use_every_xcd(tmp_path):
    out = run_plan_program(tmp_path, ORDER)
    assert out == "ok\n", out
