"""Weight gradients read straight from the gradient and the image: edges of the tiles (16 to 144 channels, weights around 128),
pixels below, at and beyond a stage, lines and images passed several times in one stage, padding and stride, one slice and many,
both tile shapes, two workgroups a CU with several stages and with slices, more slices than ride (of 64-bit sums too), and the shapes left to stored patches, 1x1 layers of few pixels among them.  Bit for bit against the CPU oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say
from tests.test_gpu_conv import check_conv, fxp  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,C,Cout,KH,KW,stride,pad", [
    (1, 1, 1, 16, 16, 1, 1, 1, 0), (1, 8, 16, 16, 64, 1, 1, 1, 0), (1, 3, 43, 32, 48, 3, 1, 1, 1), (129, 1, 1, 48, 80, 1, 1, 1, 0),
    (300, 2, 2, 16, 16, 2, 2, 1, 1), (7, 5, 3, 64, 128, 3, 3, 1, 2), (2, 17, 19, 112, 144, 3, 3, 2, 0), (3, 30, 29, 80, 64, 5, 4, 3, 2),
    (11, 14, 14, 128, 128, 3, 3, 1, 1), (12, 28, 28, 64, 64, 3, 3, 1, 1), (40, 28, 27, 16, 32, 3, 3, 1, 1), (9, 40, 1, 144, 272, 3, 1, 1, 1),
    (1, 8, 8, 512, 1024, 3, 3, 2, 1), (3, 5, 5, 512, 496, 3, 3, 1, 1), (1, 2, 2, 1024, 1024, 3, 3, 1, 1),
    (16, 7, 7, 512, 1024, 3, 3, 1, 1), (64, 14, 14, 256, 512, 3, 3, 1, 1), (4, 10, 14, 528, 1040, 3, 3, 1, 1),
    (16, 112, 112, 16, 16, 1, 1, 1, 0), (10, 103, 97, 16, 32, 1, 1, 1, 0),
    (4, 14, 14, 272, 400, 1, 1, 1, 0), (1, 56, 56, 16, 48, 1, 1, 2, 0), (20, 7, 7, 64, 80, 1, 1, 1, 0), (4, 16, 16, 32, 16, 1, 1, 1, 0),
    (1, 31, 31, 16, 80, 1, 1, 1, 0), (1, 9, 9, 24, 64, 3, 3, 1, 1), (2, 9, 9, 32, 40, 3, 3, 2, 1)])
def test_weight_gradient(fxp, N, H, W, C, Cout, KH, KW, stride, pad):  # noqa: F811
    say("weight gradient", (N, H, W, C, Cout, KH, KW, stride, pad))
    rng = np.random.default_rng(N * 1000 + H * 10 + C + Cout)
    X = rng.standard_normal((N, H, W, C)).astype(np.float32)
    Wt = rng.standard_normal((Cout, KH, KW, C)).astype(np.float32)
    Ho, Wo = oracle.conv_out_hw(H, W, KH, KW, stride, pad)
    dY = rng.laplace(0, 1e-3, (N, Ho, Wo, Cout)).astype(np.float32)
    check_conv(fxp, X, Wt, dY, stride, pad)
    check_conv(fxp, X, Wt, dY, stride, pad, bits=6, need_dX=False)
