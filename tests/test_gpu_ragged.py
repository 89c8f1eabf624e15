"""GPU parity where rows are not whole 16-byte pieces: products at the edges of the register-staged tiles and of its
contraction tail, against the CPU oracle (integers and fp32 outputs bit for bit)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, same_bits, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fxp():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: there is no CPU path in libfxp")
    from paper_2207_08822_amd import fxp as binding
    binding.lib()
    return binding


def rand_i8(rng, shape):
    return rng.integers(-127, 128, shape, dtype=np.int8)


# contraction: below one piece, one piece and a byte, around the 64- and 128-byte steps, several steps with a tail;
# outputs: one element, around 64 and 128, enough tiles for the 128 x 128 kernel (the last), split along K (2049)
@pytest.mark.parametrize("M,N,K", [(1, 1, 15), (65, 63, 16), (64, 64, 17), (63, 129, 63), (130, 66, 65), (127, 64, 127), (64, 128, 129),
                                   (129, 65, 191), (197, 70, 197), (100, 300, 385), (70, 90, 2049), (2900, 2817, 67)])
def test_gemm_rows_off_the_16_byte_grid(fxp, M, N, K):
    say("ragged gemm", (M, N, K))
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    A, B = rand_i8(rng, (M, K)), rand_i8(rng, (N, K))
    want = oracle.gemm(A, B, transB=True)
    assert np.array_equal(host(fxp.gemm(dev(A), dev(B), transB=True)), want)
    e = dev(np.array([121, 130], np.int32))
    assert same_bits(host(fxp.gemm_unmap(dev(A), dev(B), e[0:1], e[1:2], transB=True)), oracle.unmap(want, 121, 130))


@pytest.mark.parametrize("off_a,off_b", [(1, 0), (3, 7), (0, 15)])
def test_gemm_bases_off_the_16_byte_grid(fxp, off_a, off_b):
    """Operands that end with their buffer and start at any byte; K = 208 is a multiple of 16, 77 is not."""
    rng = np.random.default_rng(off_a * 16 + off_b)
    for M, N, K in [(96, 80, 208), (70, 65, 77)]:
        say("gemm unaligned bases", (off_a, off_b), (M, N, K))
        A, B = rand_i8(rng, (M, K)), rand_i8(rng, (N, K))
        da = torch.zeros(off_a + M * K, dtype=torch.int8, device="cuda")
        db = torch.zeros(off_b + N * K, dtype=torch.int8, device="cuda")
        da[off_a:] = dev(A).flatten()
        db[off_b:] = dev(B).flatten()
        got = fxp.gemm(da[off_a:].view(M, K), db[off_b:].view(N, K), transB=True)
        assert np.array_equal(host(got), oracle.gemm(A, B, transB=True))


@pytest.mark.parametrize("batch,M,N,K", [(3, 197, 64, 197), (2, 64, 197, 33), (200, 130, 129, 21), (5, 16, 16, 12)])
def test_gemm_batched_off_the_16_byte_grid(fxp, batch, M, N, K):
    say("ragged batched gemm", (batch, M, N, K))
    rng = np.random.default_rng(batch + M + K)
    A, B = rand_i8(rng, (batch, M, K)), rand_i8(rng, (batch, N, K))
    assert np.array_equal(host(fxp.gemm_batched(dev(A), dev(B))), oracle.gemm_batched(A, B, transB=True))
