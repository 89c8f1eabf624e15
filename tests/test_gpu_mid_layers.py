"""Layers between one tile a CU and a chip full of large tiles: both gradients in one launch - aligned, one of them off the 16-byte
grid, either side of the line - and forward products on quarter-size tiles, whole and partial steps.  Bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import say
from tests.test_gpu_parity import fxp, layer_check_full  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# aligned; dX off the grid; dW off the grid; a step and a piece; more than 128 large tiles forward; two per CU together and beyond
@pytest.mark.parametrize("M,K,N", [(640, 1024, 640), (688, 768, 1000), (689, 768, 1024), (1040, 1040, 80), (1100, 1152, 1100), (1616, 2000, 1600),
                                   (1616, 2000, 2960), (200, 1152, 1030), (577, 1040, 70), (130, 1104, 2050), (65, 1984, 2064)])
def test_layers_of_medium_size(fxp, M, K, N):  # noqa: F811
    say("medium layer", (M, K, N))
    rng = np.random.default_rng(M + K + N)
    layer_check_full(fxp, rng.standard_normal((M, K)).astype(np.float32), (rng.standard_normal((K, N)) * 0.1).astype(np.float32),
                     rng.laplace(0, 1e-3, (M, N)).astype(np.float32), seed=M, step=2)
