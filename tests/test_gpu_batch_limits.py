"""A batch of small and large instances, which two kernels solve: one time limit
for the whole batch, and results that do not depend on the company an instance
is solved in, over several replays of the batch's graph."""
import numpy as np
import pytest

import paper_2608_09159_amd as G
from instances import synth

pytestmark = pytest.mark.gpu


def mixed(n_small, n_large):
    ps = [synth.portfolio(1_000_000 + i, n_assets=60 + 5 * i, n_factors=5) for i in range(n_small)]
    return ps + [synth.portfolio(2_000_000 + i, n_assets=700 + 20 * i, n_factors=9) for i in range(n_large)]


def test_one_time_limit_for_the_batch():
    """No instance reaches the tolerance, so small and large ones run until the
    limit.  The device time of the call is the limit and the rest of one check
    period (64 iterations, a few milliseconds)."""
    limit = 0.4
    h = G.setup_batch(mixed(6, 6), tol=1e-300, max_iter=10 ** 9, time_limit=limit, time_kernels=1, autotune=0)
    try:
        for _ in range(2):
            res = h.solve()
            assert [r["status"] for r in res] == ["TIME_LIMIT"] * len(res)
            assert limit * 0.9 <= res[0]["kernel_s"] <= limit * 1.25, res[0]["kernel_s"]
    finally:
        h.free()


def test_company_and_replays_change_nothing():
    kw = dict(a_norm=1.0, autotune=0, max_iter=2000)
    ps = mixed(5, 4)
    alone = [G.solve(p, grid_dim=1, **kw) for p in ps]
    h = G.setup_batch(ps, **kw)
    try:
        runs = []
        for _ in range(4):
            runs.append(h.solve())
            G.project_cones("soc", np.ones((64, 5)), np.ones((64, 5)))   # other work between the replays
    finally:
        h.free()
    for res in runs:
        for r, a in zip(res, alone):
            assert r["iterations"] == a["iterations"] and r["status"] == a["status"]
            np.testing.assert_array_equal(r["x"], a["x"])
            np.testing.assert_array_equal(r["y"], a["y"])
