"""The rounding term of the fused sweep's TV bound, on the CPU: sum_P r is taken
as half of sum r plus half of sum |r| over every entry, in chains of eight
float additions that go on in double, so its rounding is a share of sum |r|,
not of sum_P r."""
import os
import re

import numpy as np

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_36601_amd", "csrc",
                      "row_engine.hpp")


def _chains(x):
    """Sums over groups of 8 in float, of the groups in double."""
    acc = np.zeros(x.size // 8, np.float32)
    for k in range(8):
        acc = (acc + x.reshape(-1, 8)[:, k]).astype(np.float32)
    return acc.astype(np.float64).sum()


def test_the_bound_covers_the_rounding_of_the_halves():
    with open(HEADER) as f:
        share = float(re.search(r"FUSED_SUM_ROUND = ([0-9.e-]+);", f.read()).group(1))
    rng = np.random.default_rng(0)
    worst_all = worst_p = 0.0
    for _ in range(1500):
        V = 1024 * int(rng.integers(1, 6))
        s = rng.normal(0, rng.uniform(0.5, 5.0), V)
        t = 0.6 * s + rng.normal(0, rng.uniform(0.3, 3.0), V)
        lp, lt = s - np.log(np.exp(s).sum()), t - np.log(np.exp(t).sum())
        x = rng.uniform(0.05, 1.0) * (lt - lp)
        y = (x - np.log(np.exp(lp + x).sum())).astype(np.float32).astype(np.float64)
        pt = np.exp(lp - lp.max()).astype(np.float32)
        r = (pt * np.expm1(y)).astype(np.float32)
        t0 = 0.5 * (_chains(r) + _chains(np.abs(r)))
        pos, both = np.maximum(r.astype(np.float64), 0.0).sum(), np.abs(r.astype(np.float64)).sum()
        worst_all = max(worst_all, abs(t0 - pos) / both)
        worst_p = max(worst_p, abs(t0 - pos) / pos)
    assert worst_all < share
    assert worst_p > 1e-7  # the share of sum_P r that the bound once allowed
