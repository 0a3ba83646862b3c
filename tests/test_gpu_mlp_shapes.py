"""The network's products at the edges of their kernels: tiles of 32, 64 and
128, up to 32 rows and one past, one chunk of K and several, chunks spread over
workgroups (one row, long K), odd leading dimensions (elementwise loads), and
contiguous dimensions that end 2 into a run of 4 or are shorter than one.

Exact regime (see test_gpu_mlp): every forward sum is exact, so the forward pass
and the loss agree with the FP64 reference bit for bit.  Gradients: the FP32
accumulation bound plus one BF16 step of the backward signals."""
import numpy as np
import pytest

import test_gpu_mlp as T
from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,B", [
    ([3000, 33, 65, 31], 1),         # one row, 47 steps of K spread over workgroups
    ([2, 3, 1, 2], 2),               # shorter than a run
    ([1030, 64, 32, 66], 31),        # up to 32 rows, K 6 past a step
    ([130, 65, 63, 129], 32),        # odd leading dimensions
    ([64, 62, 66, 130], 33),         # one row past: staged or a wave per chunk
    ([1025, 34, 70, 514], 65),
    ([700, 514, 258, 1026], 130),    # many 64 x 64 tiles, several chunks
    ([66, 2050, 130, 3074], 250),
])
def test_products_at_tile_edges(dims, B):
    rng = np.random.default_rng(sum(dims) + B)
    Ws, bs, X, Y = T._exact_case(rng, dims, B)
    ref = M.MLP(Ws, bs)
    T._exact_precondition(ref, X)
    net = T._net(dims, B, Ws, bs)
    try:
        yh = net.forward(T._dev(X)).cpu().numpy().astype(np.float64)
        loss = net.train_step(T._dev(X), T._dev(Y), update=False)
        grads = [net.grads(k) for k in range(len(Ws))]
    finally:
        net.free()
    np.testing.assert_array_equal(yh, ref.forward(X)[0])
    rloss, rdW, rdb, dzs, hs = ref.gradients(X, Y, signals=True)
    assert loss == pytest.approx(rloss, rel=1e-12)
    for k in range(len(Ws)):
        bound = (2.0 ** -7 + B * 2.0 ** -24) * (np.abs(hs[k]).T @ np.abs(dzs[k]))
        assert np.all(np.abs(grads[k][0] - rdW[k]) <= bound), k
        bound = (2.0 ** -7 + B * 2.0 ** -24) * np.abs(dzs[k]).sum(axis=0)
        assert np.all(np.abs(grads[k][1] - rdb[k]) <= bound), k
