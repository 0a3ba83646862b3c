"""A solve whose workgroups stop waiting for each other (settings.verbose bit 4:
waits of one clock tick) ends as ABORTED on every core that runs on a grid,
and leaves nothing behind: the next solves are those of a fresh handle."""
import numpy as np
import pytest

import paper_2608_09159_amd as G
from instances import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(grid_dim=4), dict(grid_dim=4, scheme=1), dict(grid_dim=4, precision=1)])
def test_short_waits_end_as_aborted(kw):
    p = synth.tiny_qp(2)
    r = G.solve(p, max_iter=200, **kw)
    a = G.solve(p, max_iter=200, verbose=16, **kw)
    assert a["status"] == "ABORTED"
    b = G.solve(p, max_iter=200, **kw)
    assert b["status"] == r["status"] != "ABORTED"
    np.testing.assert_array_equal(b["x"], r["x"])


def test_one_workgroup_waits_for_nobody():
    p = synth.tiny_qp(2)
    assert G.solve(p, max_iter=200, grid_dim=1, verbose=16)["status"] != "ABORTED"
