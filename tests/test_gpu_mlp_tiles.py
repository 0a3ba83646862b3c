"""Which way a product of the network goes: tiles of 128 in one turn of the chip
and in two, tiles of 64 for one chunk of K and for several, and long sums over K
whose chunks travel through memory (K inside a chunk at the end), for both
layouts of the right operand.

Exact regime (see test_gpu_mlp): every forward sum is exact, so the forward
pass and the loss agree with the FP64 reference bit for bit.  Gradients: a
backward signal is off by one BF16 step of its own, by the FP32 accumulation
of its product and by what the next layer's signal was off; the weight
gradient by these and by its own accumulation over the batch."""
import numpy as np
import pytest

import test_gpu_mlp as T
from oracle import mlp as M

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.mark.parametrize("dims,B", [
    ([16, 24, 49000], 256),      # 766 tiles of 128: one turn
    ([16, 24, 49000], 385),      # 1,532 tiles: two turns
    ([16, 24, 50002], 250),      # 782 tiles: just a second turn
    ([16, 24, 40002], 129),      # 626 tiles, the last row almost empty
    ([16, 24, 33001], 192),      # odd leading dimension
    ([16, 24, 33000], 257),      # 774 tiles, the last row almost empty
    ([64, 520, 24], 200),        # one step of K, fewer tiles than CUs
    ([16, 49000, 24], 256),      # the transposed product over 49,000 columns
    ([6100, 48, 40], 40),        # K beyond 6,000, inside a chunk at the end
    ([7000, 130, 33], 130),
    ([40, 48, 6500], 40),        # the same for the transposed product
    ([33, 130, 7002], 200),
    ([2050, 2602, 30], 260),     # several chunks, ragged in every direction: through memory
    ([1029, 2601, 33], 129),     # the same in single elements
    ([130, 9002, 34], 300),      # two chunks, tiles of 64
])
def test_products_by_tile(dims, B):
    print(f"[tiles] {dims} batch {B}", flush=True)
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
    err = np.zeros_like(dzs[-1])
    for k in reversed(range(len(Ws))):
        z = np.abs(dzs[k])
        if k < len(Ws) - 1:
            W = np.abs(M.bf16_round(Ws[k + 1]))
            err = err @ W.T + dims[k + 2] * U * (np.abs(dzs[k + 1]) @ W.T)
        err = err + 2.0 ** -7 * z
        h = np.abs(hs[k])
        assert np.all(np.abs(grads[k][0] - rdW[k]) <= h.T @ (err + B * U * z)), k
        assert np.all(np.abs(grads[k][1] - rdb[k]) <= (err + B * U * z).sum(axis=0)), k
