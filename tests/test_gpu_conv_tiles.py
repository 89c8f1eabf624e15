"""Tiles of implicit convolutions.  Input gradients of stride-2 convolutions, computed per class of input pixels: odd and even sizes, filters smaller than
the stride (classes without taps), paddings beyond the filter, rows and columns that no output reads, one image row per
class, several tiles per class, both K steps, and the weight gradient's sum riding along.  Bit for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say
from tests.test_gpu_conv import check_conv, fxp  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

CASES = [  # N, H, W, C, Cout, KH, KW, pad
    (2, 8, 8, 32, 64, 3, 3, 1), (2, 9, 7, 32, 64, 3, 3, 1), (1, 11, 12, 33, 128, 3, 3, 0), (3, 8, 9, 64, 128, 1, 1, 0),
    (2, 7, 8, 40, 64, 1, 1, 1), (1, 6, 5, 48, 192, 1, 3, 2), (2, 10, 10, 36, 64, 2, 2, 0), (1, 13, 9, 64, 64, 5, 4, 3),
    (1, 12, 15, 32, 64, 7, 7, 3), (1, 1, 9, 64, 128, 1, 3, 1), (1, 3, 2, 130, 128, 3, 2, 0),
    (3, 29, 27, 129, 128, 3, 3, 1), (12, 28, 28, 128, 256, 3, 3, 1), (44, 28, 28, 128, 128, 3, 3, 1), (17, 33, 32, 64, 128, 3, 3, 1)]


def _tensors(N, H, W, C, Cout, KH, KW, pad):
    rng = np.random.default_rng(N * 1000 + H * 10 + C)
    X = rng.standard_normal((N, H, W, C)).astype(np.float32)
    Wt = rng.standard_normal((Cout, KH, KW, C)).astype(np.float32)
    Ho, Wo = oracle.conv_out_hw(H, W, KH, KW, 2, pad)
    return X, Wt, rng.laplace(0, 1e-3, (N, Ho, Wo, Cout)).astype(np.float32)


@pytest.mark.parametrize("N,H,W,C,Cout,KH,KW,pad", CASES)
def test_strided_input_gradient(fxp, N, H, W, C, Cout, KH, KW, pad):  # noqa: F811
    say("strided conv", (N, H, W, C, Cout, KH, KW, pad))
    check_conv(fxp, *_tensors(N, H, W, C, Cout, KH, KW, pad), 2, pad)


@pytest.mark.parametrize("N,H,W,C,Cout,KH,pad", [
    (3, 14, 14, 128, 256, 3, 1), (2, 7, 7, 512, 512, 3, 1), (5, 9, 11, 192, 320, 3, 0), (70, 14, 13, 64, 256, 3, 1),
    (1, 5, 5, 128, 65, 1, 0), (90, 14, 14, 256, 256, 3, 1), (2, 9, 8, 24, 40, 1, 0), (64, 28, 14, 128, 256, 1, 0), (43, 28, 28, 128, 128, 3, 1)])
def test_few_tiles(fxp, N, H, W, C, Cout, KH, pad):  # noqa: F811
    """Stride 1: the quarter-size tiles of small outputs (at most 128 large ones), either K step, and both sides of the
    rule; more tiles than CUs; 1x1 layers whose patches are the image itself."""
    say("conv, few tiles", (N, H, W, C, Cout, KH, pad))
    rng = np.random.default_rng(N * 1000 + H * 10 + C)
    X = rng.standard_normal((N, H, W, C)).astype(np.float32)
    Wt = rng.standard_normal((Cout, KH, KH, C)).astype(np.float32)
    Ho, Wo = oracle.conv_out_hw(H, W, KH, KH, 1, pad)
    check_conv(fxp, X, Wt, rng.laplace(0, 1e-3, (N, Ho, Wo, Cout)).astype(np.float32), 1, pad)


# down to 8 channels, and the 7 below
@pytest.mark.parametrize("N,H,W,C,Cout,KH,KW,pad", [(3, 15, 14, 8, 64, 3, 3, 1), (2, 14, 17, 7, 64, 3, 3, 1), (40, 28, 27, 9, 64, 5, 5, 2),
                                                    (5, 31, 30, 24, 128, 3, 3, 0), (2, 20, 20, 31, 192, 2, 3, 1), (6, 28, 28, 16, 64, 1, 1, 0)])
def test_strided_input_gradient_of_few_channels(fxp, N, H, W, C, Cout, KH, KW, pad):  # noqa: F811
    say("strided conv, few channels", (N, H, W, C, Cout, KH, KW, pad))
    check_conv(fxp, *_tensors(N, H, W, C, Cout, KH, KW, pad), 2, pad)


@pytest.mark.parametrize("case", [CASES[1], CASES[4], CASES[11]])
def test_strided_input_gradient_alone(fxp, case):  # noqa: F811
    say("strided conv, dX alone", case)
    check_conv(fxp, *_tensors(*case), 2, case[-1], bits=5, need_dW=False)


# more than 128 large tiles and at most 64 output channels: 128 x 64 tiles, ragged in the last row tile and in the columns
@pytest.mark.parametrize("N,H,W,C,Cout,KH", [(6, 53, 53, 64, 64, 3), (6, 53, 53, 64, 64, 1), (6, 53, 53, 64, 40, 3), (5, 59, 57, 192, 8, 3)])
def test_many_tiles_of_few_channels(fxp, N, H, W, C, Cout, KH):  # noqa: F811
    say("conv, 128 x 64 tiles", (N, H, W, C, Cout, KH))
    rng = np.random.default_rng(H + C + Cout)
    X = np.maximum(rng.standard_normal((N, H, W, C)), 0).astype(np.float32)
    Wt = rng.standard_normal((Cout, KH, KH, C)).astype(np.float32)
    assert N * H * W > 128 * 128
    check_conv(fxp, X, Wt, rng.laplace(0, 1e-3, (N, H, W, Cout)).astype(np.float32), 1, KH // 2)


# both sides of the rule on long contractions in few tiles: 5184 terms over 16 and 49 pixels, 9216 over 64 and 98, beyond
# 18432; 1x1 layers around 2048 channels
@pytest.mark.parametrize("N,H,C,Cout,KH", [(1, 4, 576, 64, 3), (1, 7, 576, 64, 3), (1, 8, 1024, 70, 3), (2, 7, 1024, 64, 3), (3, 8, 2112, 64, 3),
                                           (2, 7, 2048, 100, 1), (2, 7, 2112, 128, 1), (2, 7, 128, 2112, 1)])
def test_long_contractions_in_few_tiles(fxp, N, H, C, Cout, KH):  # noqa: F811
    say("conv, long contraction, few tiles", (N, H, C, Cout, KH))
    rng = np.random.default_rng(H + C + Cout)
    X = np.maximum(rng.standard_normal((N, H, H, C)), 0).astype(np.float32)
    Wt = rng.standard_normal((Cout, KH, KH, C)).astype(np.float32)
    check_conv(fxp, X, Wt, rng.laplace(0, 1e-3, (N, H, H, Cout)).astype(np.float32), 1, KH // 2)


# both sides of the rule on the longest class of a strided input gradient: 512 and 1024 channels (2048 and 4096 terms), few
# tiles (patch gradient) and enough of them (classes); beyond 4096 terms
@pytest.mark.parametrize("N,H,C,Cout,KH", [(2, 14, 64, 512, 3), (19, 14, 129, 512, 3), (2, 9, 33, 1024, 3), (37, 14, 257, 1024, 3), (3, 9, 32, 1088, 3),
                                           (2, 12, 64, 2112, 1)])
def test_strided_input_gradient_long_classes(fxp, N, H, C, Cout, KH):  # noqa: F811
    say("strided conv, long classes", (N, H, C, Cout, KH))
    pad = KH // 2
    check_conv(fxp, *_tensors(N, H, H, C, Cout, KH, KH, pad), 2, pad)
