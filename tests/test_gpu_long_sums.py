"""GPU parity of weight gradients over more rows or pixels than one int32 sum holds (133 144), whose slices are added in 64
bits: in a launch of their own or riding in the input gradient's, with tails and outputs off the 16-byte grid, bit for bit
against the oracle.  Column 0 and channel 0 are at the top code everywhere, so those sums pass 2^31."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, same_bits, say
from tests.test_gpu_conv import check_conv, fxp  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# dX a register-staged product (ragged K and N, outputs with a tail), a direct-to-LDS one, and none
@pytest.mark.parametrize("M,K,N,need_dX", [(133160, 33, 65, True), (140000, 128, 64, True), (133145, 40, 24, False)])
@pytest.mark.parametrize("offset", [0, 1])
def test_linear(fxp, M, K, N, need_dX, offset):  # noqa: F811
    """offset: dW starts that many elements behind a 16-byte boundary."""
    say("linear, long sums", (M, K, N), "dX" if need_dX else "no dX", "offset", offset)
    rng = np.random.default_rng(M + K)
    X = rng.standard_normal((M, K)).astype(np.float32).clip(-3.9, 3.9)
    W = (rng.standard_normal((K, N)) * 0.1).astype(np.float32)
    dY = rng.uniform(-1e-3, 1e-3, (M, N)).astype(np.float32)
    X[:, 0], dY[:, 0] = 127 / 32, 127 * 2.0 ** -16             # top code in every row (units 2^-5 and 2^-16)
    buf = fxp.LayerBuffers(M, K, N)
    room = torch.zeros(K * N + 8, device="cuda")
    buf.dW = room[offset:offset + K * N].view(K, N)
    fxp.linear_fwd(dev(X), dev(W), buf, seed=2, step=3)
    dX, dW = fxp.linear_bwd(dev(dY), buf, seed=2, step=3, need_dX=need_dX)
    _, saved = oracle.linear_fwd(X, W, seed=2, step=3)
    dXo, dWo, _ = oracle.linear_bwd(dY, saved, seed=2, step=3)
    assert same_bits(host(dW), dWo)
    assert dX is None or same_bits(host(dX), dXo)
    assert not host(room[:offset]).any() and not host(room[offset + K * N:]).any()


# the gradient read from the image (C and Cout multiples of 16), of stride 1 and 2, and of a 1x1 layer; stored patches (C = 20 and 36)
# with the sum riding in an implicit input gradient of stride 1 and of stride 2, launched before one of stored patches, and alone
@pytest.mark.parametrize("N,H,W,C,Cout,KH,stride,pad,need_dX", [
    (3, 212, 212, 16, 16, 3, 1, 1, True), (3, 211, 212, 20, 64, 3, 1, 1, True), (2, 519, 520, 32, 64, 3, 2, 1, True), (43, 56, 56, 64, 64, 1, 1, 0, True),
    (2, 519, 520, 20, 64, 3, 2, 1, True), (3, 211, 212, 36, 24, 3, 1, 1, True), (3, 211, 212, 20, 64, 3, 1, 1, False), (2, 519, 520, 36, 64, 3, 2, 1, False)])
def test_conv(fxp, N, H, W, C, Cout, KH, stride, pad, need_dX):  # noqa: F811
    say("conv, long sums", (N, H, W, C, Cout, KH, stride, pad), "dX" if need_dX else "no dX")
    rng = np.random.default_rng(H + C)
    X = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0).clip(0, 3.9)
    Wt = rng.standard_normal((Cout, KH, KH, C), dtype=np.float32) * np.float32(0.1)
    Ho, Wo = oracle.conv_out_hw(H, W, KH, KH, stride, pad)
    assert N * Ho * Wo > 133144
    dY = rng.uniform(-1e-3, 1e-3, (N, Ho, Wo, Cout)).astype(np.float32)
    X[..., 0], dY[..., 0] = 127 / 32, 127 * 2.0 ** -16
    check_conv(fxp, X, Wt, dY, stride, pad, need_dX=need_dX)
