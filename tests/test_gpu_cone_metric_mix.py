"""Blocks of constant and of varying metric side by side in one wave: the
projection kernel tells them apart by itself, a group of 16, 32 or 64 lanes a
block.  Dimensions at the edges of those groups; the metric of every third
block is constant, that of every fourth differs in its last coordinate alone.

Tolerance: 1e-9 max(1, ||r||_inf) a block, that of the projections against the
oracle at large."""
import numpy as np
import pytest

import paper_2608_09159_amd as G
from oracle import cones as OC

pytestmark = pytest.mark.gpu

TOL = 1e-9


@pytest.mark.parametrize("dim", [2, 3, 16, 17, 18, 32, 33, 34, 63, 64, 65, 66, 130])
@pytest.mark.parametrize("kind", ["soc", "rsoc"])
def test_constant_and_varying_metrics_in_one_wave(kind, dim):
    rng = np.random.default_rng(dim)
    n = 203
    R = rng.standard_normal((n, dim)) * 10.0 ** rng.uniform(-2, 2, (n, 1))
    M = 10.0 ** rng.uniform(-1, 1, (n, dim))
    M[::3] = M[::3, :1]
    M[::4, :-1] = M[::4, :1]
    dev = G.project_cones(kind, R, M)
    ref = (OC.soc_metric if kind == "soc" else OC.rsoc_metric)(R, M)
    err = np.max(np.abs(dev - ref), axis=1) / np.maximum(1.0, np.max(np.abs(R), axis=1))
    assert np.max(err) <= TOL
