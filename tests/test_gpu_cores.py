"""Which core solves a problem (the last column of PDHCG_PARTITION_DUMP: 0 the
general core, 1 and 2 the register-resident grid core with one and two
coordinates and rows a thread, 3 the same on one workgroup), and the general
core on a grid at sizes that the resident core does not take: lane mappings,
length classes, bounds and boxes with cone blocks and without.  Then the resident
core's edges with bounds, boxes and fixed-middle EXP blocks.

Tolerance: that of the other parity tests (1e-10 relative on the first
iterations, counts and decisions exactly)."""
import os

import numpy as np
import pytest
import scipy.sparse as sp

import paper_2608_09159_amd as G
from instances import Problem, synth
from parity_util import trace_parity

pytestmark = pytest.mark.gpu

GENERAL, ONE_EACH, TWO_EACH, ONE = 0, 1, 2, 3


def parity_on(core, prob, tmp_path, iters=30, **kw):
    path = str(tmp_path / "partition.txt")
    os.environ["PDHCG_PARTITION_DUMP"] = path
    try:
        G.setup(prob, **kw).free()
    finally:
        del os.environ["PDHCG_PARTITION_DUMP"]
    assert set(np.loadtxt(path, dtype=np.int64, ndmin=2)[:, 8]) == {core}
    trace_parity(prob, iters=iters, **kw)


# ---------------------------------------------------------------- general core
@pytest.mark.parametrize("lanes", [1, 2, 16, 64])
def test_lane_mappings(lanes, tmp_path):
    p = synth.fisher(seed=5, n_buyers=500, n_goods=40, density=0.25)
    assert p.n > 3 * 1024
    parity_on(GENERAL, p, tmp_path, lanes_at=lanes, lanes_a=lanes, grid_dim=3)


def test_two_lane_counts(tmp_path):
    p = synth.large_sparse_qp(seed=3, n=6_000, m=3_000)
    parity_on(GENERAL, p, tmp_path, lanes_at=4, lanes_a=2, grid_dim=3)


@pytest.mark.parametrize("grid", [3, 16])
def test_mixed_cones(grid, tmp_path):
    parity_on(GENERAL, synth.mixed_cone_scaled(seed=4, scale=0.2), tmp_path, iters=20, grid_dim=grid)


def test_skewed_columns(tmp_path):
    """Power-law column degrees: the longest A^T rows get workgroups of their
    own and the others run in length classes."""
    p = synth.large_sparse_qp(seed=1, n=60_000, m=30_000)
    parity_on(GENERAL, p, tmp_path, iters=20, grid_dim=24)


@pytest.mark.parametrize("q", ["lowrank", "diag", None])
@pytest.mark.parametrize("cones", [True, False])
def test_bounds_on_a_grid(q, cones, tmp_path):
    p = synth.bounded_qp(13, n_box=4000, n_cone_soc=40 if cones else 0, n_exp=20 if cones else 0, m=900,
                         density=0.004, q=q)
    parity_on(GENERAL, p, tmp_path, grid_dim=3)


def test_long_rows_leave_the_resident_core(tmp_path):
    rng = np.random.default_rng(1)
    n = 100
    A = sp.csr_matrix(rng.standard_normal((n, n)) / 10)
    p = Problem(n=n, m=n, A=A, b=A @ rng.random(n), c=rng.standard_normal(n), P=sp.identity(n, format="csr"), R=None,
                D=None, cones=[("nonneg", 0, n, 0.0)], name="dense")
    parity_on(GENERAL, p, tmp_path, grid_dim=1)


# --------------------------------------------------------------- resident core
@pytest.mark.parametrize("n_box,m,grid,core,q,soc,exp", [
    (503, 512, 1, ONE, "diag", 0, 0),          # 512 coordinates and rows
    (474, 300, 1, ONE, "lowrank", 4, 3),       # 512 with cone blocks
    (700, 600, 2, ONE_EACH, "lowrank", 0, 0),  # the ranges are cut by work, not by count
    (1800, 1500, 2, TWO_EACH, "lowrank", 0, 0),
    (1600, 1300, 2, TWO_EACH, "diag", 5, 4),
    (450, 400, 2, ONE_EACH, None, 8, 10),
])
def test_bounds_at_the_edges(n_box, m, grid, core, q, soc, exp, tmp_path):
    p = synth.bounded_qp(n_box + m, n_box=n_box, n_cone_soc=soc, n_exp=exp, m=m, density=8.0 / n_box, q=q)
    parity_on(core, p, tmp_path, grid_dim=grid)


def fixed_middle(buyers, goods, per):
    """A market of the paper's shape at any size: synth.fisher_paper's blocks."""
    return synth.fisher(seed=9, n_buyers=buyers, n_goods=goods, density=per, middle="fixed")


@pytest.mark.parametrize("buyers,goods,density,grid,core", [
    (60, 20, 0.1, 1, ONE),
    (60, 20, 0.1, 2, ONE_EACH),
    (150, 60, 0.06, 2, TWO_EACH),
    (500, 60, 0.08, 2, GENERAL),
])
def test_fixed_middle_blocks(buyers, goods, density, grid, core, tmp_path):
    parity_on(core, fixed_middle(buyers, goods, density), tmp_path, grid_dim=grid)
