"""GPU parity of convolutions over a few channels (the image itself), whose kernels read the image directly: edges of the
32-pixel tiles and 16-pixel pieces, of the 32-byte filter rows, of the channel fragments and of the units of output rows,
against the CPU oracle bit for bit; and the sum of many slices of a small output."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, same_bits, say
from tests.test_gpu_conv import check_conv, fxp  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [  # N, H, W, C, Cout, KH, KW, stride, pad
    (1, 1, 1, 3, 1, 1, 1, 1, 0), (2, 3, 5, 1, 33, 3, 3, 2, 1), (1, 9, 33, 3, 64, 7, 7, 2, 3), (3, 40, 31, 3, 64, 7, 7, 2, 3),
    (2, 17, 34, 4, 96, 3, 3, 2, 1), (2, 16, 16, 4, 128, 7, 8, 1, 3), (1, 20, 47, 2, 32, 5, 16, 3, 8), (4, 33, 63, 3, 65, 3, 3, 1, 1),
    (1, 70, 18, 1, 97, 9, 7, 4, 0), (2, 12, 13, 4, 31, 11, 1, 2, 5), (1, 30, 6, 3, 40, 3, 6, 5, 2), (1, 8, 9, 4, 8, 3, 9, 1, 1),
    (1, 12, 12, 3, 130, 3, 3, 1, 1), (40, 35, 37, 3, 16, 3, 3, 2, 1), (600, 4, 4, 1, 4, 3, 3, 1, 1)]


@pytest.mark.parametrize("N,H,W,C,Cout,KH,KW,stride,pad", CASES)
def test_thin_conv(fxp, N, H, W, C, Cout, KH, KW, stride, pad):  # noqa: F811
    say("thin conv", (N, H, W, C, Cout, KH, KW, stride, pad))
    rng = np.random.default_rng(N * 1000 + H * 10 + W)
    X = rng.standard_normal((N, H, W, C)).astype(np.float32)
    Wt = (rng.standard_normal((Cout, KH, KW, C)) * 0.1).astype(np.float32)
    Ho, Wo = oracle.conv_out_hw(H, W, KH, KW, stride, pad)
    dY = rng.laplace(0, 1e-3, (N, Ho, Wo, Cout)).astype(np.float32)
    check_conv(fxp, X, Wt, dY, stride, pad, need_dX=False)
    if N < 10:
        check_conv(fxp, X, Wt, dY, stride, pad, rounding=1, bits=5)


# many units of few pixels, on both sides of the line between transposed patches and the image itself
@pytest.mark.parametrize("N,H,W,C,Cout,KH,KW", [(900, 2, 2, 1, 33, 2, 2), (700, 4, 4, 1, 16, 1, 1), (700, 4, 4, 3, 16, 3, 1),
                                                (600, 5, 5, 3, 130, 3, 3), (600, 5, 5, 3, 128, 3, 3), (600, 5, 5, 3, 31, 3, 3),
                                                (5, 4096, 1, 4, 64, 3, 1), (5, 4096, 1, 2, 16, 5, 1), (40, 300, 1, 1, 16, 3, 1),
                                                (700, 3, 5, 4, 64, 3, 3), (20, 256, 16, 4, 32, 3, 3), (9, 512, 8, 1, 128, 1, 1)])
def test_many_small_units(fxp, N, H, W, C, Cout, KH, KW):  # noqa: F811
    say("thin conv, small units", (N, H, W, C, Cout, KH, KW))
    rng = np.random.default_rng(N + H + W)
    X = rng.standard_normal((N, H, W, C)).astype(np.float32)
    Wt = (rng.standard_normal((Cout, KH, KW, C)) * 0.1).astype(np.float32)
    dY = rng.laplace(0, 1e-3, (N, H - KH + 1, W - KW + 1, Cout)).astype(np.float32)
    check_conv(fxp, X, Wt, dY, 1, 0)


def test_thin_conv_beyond_one_int32_sum(fxp):  # noqa: F811
    """136 161 output pixels of one sign: the slices need 64 bits together."""
    say("thin conv, long contraction")
    X = np.ones((9, 245, 245, 1), np.float32)
    Wt = np.full((3, 3, 3, 1), 0.5, np.float32)
    dY = np.full((9, 123, 123, 3), 1.99, np.float32)
    check_conv(fxp, X, Wt, dY, 2, 1, need_dX=False)


# outputs: pieces short of one wave, a tail of 3, not flat is impossible here (dense); slices: 15, 16, 17 and many
@pytest.mark.parametrize("M,N,K", [(5, 7, 16400), (8, 8, 17000), (64, 147, 40000), (33, 31, 100000), (3, 5, 150000), (128, 130, 33000)])
def test_sum_of_many_slices(fxp, M, N, K):  # noqa: F811
    say("many slices", (M, N, K))
    rng = np.random.default_rng(M + N + K)
    A, B = (rng.integers(-127, 128, (r, K), dtype=np.int8) for r in (M, N))
    e = dev(np.array([121, 130], np.int32))
    want = A.astype(np.int64) @ B.astype(np.int64).T
    if K <= 133144:
        want = oracle.unmap(want.astype(np.int32), 121, 130)
    else:
        want = np.ldexp(want.astype(np.float64), (121 - 133) + (130 - 133)).astype(np.float32)
    assert same_bits(host(fxp.gemm_unmap(dev(A), dev(B), e[0:1], e[1:2], transB=True)), want)
