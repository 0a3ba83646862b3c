"""The register-resident solver core at the edges of what it holds, and the
general core one step past them, against the oracle iteration by iteration.

One workgroup holds up to 512 coordinates and rows; on a grid a workgroup holds
up to 512 of each one a thread, or up to 1,024 two a thread.  Rows of more than
32 entries are summed by a wave; products are staged 4,096 at a time; the
columns of R lie in LDS where they fit (at 32 x 512 they do not beside 4,096
products).  A short polling interval makes the launch save and reload its state.

Tolerance: the trace tolerance of the other parity tests (1e-10 relative)."""
import numpy as np
import pytest
import scipy.sparse as sp

from instances import Problem, synth
from parity_util import trace_parity

pytestmark = pytest.mark.gpu


def make(seed, n, m, q, row, cones):
    """n coordinates, m rows of `row` entries and one of n / 2; Q diagonal,
    sparse, or diagonal plus rank r ("rank8")."""
    rng = np.random.default_rng(seed)
    spec, st = [], 0
    if cones:
        for kind, d, al in (("soc", 40, 0.0), ("exp", 3, 0.0), ("pow", 3, 0.4), ("rsoc", 5, 0.0)) * 3:
            spec.append((kind, st, d, al))
            st += d
    spec.append(("nonneg", st, n - st, 0.0))
    rows, cols = [], []
    for i in range(m):
        k = n // 2 if i == m // 2 else min(row, n)
        rows.append(np.full(k, i))
        cols.append(np.sort(rng.choice(n, k, replace=False)))
    if m:
        rows, cols = np.concatenate(rows), np.concatenate(cols)
        A = sp.csr_matrix((rng.standard_normal(rows.size) / np.sqrt(row), (rows, cols)), shape=(m, n))
    else:
        A = sp.csr_matrix((0, n))
    P = sp.diags(rng.uniform(0.1, 1.0, n)).tocsr()
    R = D = None
    if q == "sparse":
        B = sp.random(n, n, 3.0 / n, random_state=rng, data_rvs=rng.standard_normal, format="csr")
        P = (P + 0.1 * (B.T @ B)).tocsr()
    elif q.startswith("rank"):
        r = int(q[4:])
        R, D = rng.standard_normal((r, n)) / np.sqrt(n), np.eye(r)
    return Problem(n=n, m=m, A=A, b=A @ synth._interior_point(rng, n, spec), c=rng.standard_normal(n), P=P, R=R, D=D,
                   cones=spec, name=f"resident[{n},{m},{q},{row},{cones}]")


@pytest.mark.parametrize("n,m,grid,q,row,cones,poll", [
    (512, 512, 1, "sparse", 4, False, 512),
    (512, 512, 1, "rank8", 4, True, 7),
    (511, 64, 1, "diag", 120, False, 512),
    (513, 300, 1, "rank8", 4, True, 512),
    (300, 513, 1, "sparse", 4, False, 512),
    (1024, 1000, 2, "rank8", 4, True, 7),
    (1024, 40, 2, "rank32", 120, False, 512),
    (1026, 800, 2, "diag", 4, True, 512),
    (2048, 2048, 2, "sparse", 5, False, 7),
    (2048, 1500, 2, "diag", 5, False, 512),
    (2060, 100, 2, "rank8", 60, True, 512),
    (700, 0, 2, "diag", 1, True, 512),
])
def test_edges_of_the_resident_core(n, m, grid, q, row, cones, poll):
    trace_parity(make(n + m, n, m, q, row, cones), iters=30, grid_dim=grid, host_poll=poll)
