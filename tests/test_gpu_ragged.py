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


# columns: the narrowest the tiles take, around 64 and 128 at every residue of 4, two column tiles; rows: one, around the
# 16-byte pieces of the transposed copy and the tile heights; the last reaches the four-pass tiles
@pytest.mark.parametrize("rows,cols", [(1, 17), (15, 63), (17, 65), (33, 66), (64, 127), (130, 129), (257, 131), (40, 190), (300, 197),
                                       (70, 15), (128, 256), (129, 260), (5000, 3), (66000, 65), (17000, 1001)])
@pytest.mark.parametrize("offset", [0, 1])
def test_map_rows_off_the_quad_grid(fxp, rows, cols, offset):
    """Both copies from x and q that start on or off the 16-byte grid, a value that saturates, one above the scale, Inf
    and NaN among them; then the row-major copy alone (the flat path)."""
    say("ragged map", (rows, cols), "offset", offset)
    rng = np.random.default_rng(rows * 131 + cols)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    e = oracle.scale(x)
    x.flat[rng.integers(0, x.size, 6)] = np.array([np.inf, -np.inf, np.nan, 1e30, 1.9999999 * 2.0 ** (e - 127), 1e-42], np.float32)
    want = oracle.map(x, e, seed=5, stream_id=77)
    n = rows * cols
    xd = torch.zeros(n + offset, dtype=torch.float32, device="cuda")
    xd[offset:] = dev(x).flatten()
    q = torch.zeros(n + 3 * offset, dtype=torch.int8, device="cuda")
    qT = torch.zeros(n + 5 * offset, dtype=torch.int8, device="cuda")
    ed = dev(np.array([e], np.int32))
    p = lambda t: t.data_ptr()
    args = (p(ed), p(q) + 3 * offset, p(qT) + 5 * offset)
    assert fxp.lib().fxp_map(p(xd) + 4 * offset, rows, cols, *args, 5, 77, 0, 8, None) == 0
    torch.cuda.synchronize()
    assert np.array_equal(host(q)[3 * offset:].reshape(rows, cols), want)
    assert np.array_equal(host(qT)[5 * offset:].reshape(cols, rows), want.T)
    q.zero_()
    assert fxp.lib().fxp_map(p(xd) + 4 * offset, rows, cols, p(ed), p(q) + 3 * offset, None, 5, 77, 0, 8, None) == 0
    torch.cuda.synchronize()
    assert np.array_equal(host(q)[3 * offset:].reshape(rows, cols), want)
    assert not host(q)[:3 * offset].any()


# products of at most one 32 x 32 tile per CU and at most 1024 terms: tile edges, contractions of one piece up to the
# longest, every residue of the 32-byte steps over the four waves; and the sizes just beyond
@pytest.mark.parametrize("M,N,K", [(1, 1, 16), (31, 33, 17), (32, 32, 32), (64, 64, 128), (33, 65, 159), (256, 256, 256), (512, 512, 1024),
                                   (511, 513, 96), (1, 4096, 1023), (70, 31, 1024), (70, 31, 1025), (520, 520, 64)])
def test_small_gemm(fxp, M, N, K):
    say("small gemm", (M, N, K))
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    A, B = rand_i8(rng, (M, K)), rand_i8(rng, (N, K))
    want = oracle.gemm(A, B, transB=True)
    assert np.array_equal(host(fxp.gemm(dev(A), dev(B), transB=True)), want)
    e = dev(np.array([3, 5], np.int32))                               # a sub-normal unit
    assert same_bits(host(fxp.gemm_unmap(dev(A), dev(B), e[0:1], e[1:2], transB=True)), oracle.unmap(want, 3, 5))
    absmax = torch.zeros(fxp.ABSMAX_WORDS, dtype=torch.int32, device="cuda")
    C = host(fxp.gemm_unmap_absmax(dev(A), dev(B), dev(np.array([121], np.int32)), dev(np.array([130], np.int32)), absmax, transB=True))
    assert same_bits(C, oracle.unmap(want, 121, 130))
    assert int(host(absmax).max()) == int(np.abs(C).max().view(np.uint32))


# both gradients of a layer in one launch: small products, register-staged ones (odd rows), one of each kind (two launches)
@pytest.mark.parametrize("M,K,N", [(32, 64, 64), (256, 256, 256), (100, 96, 64), (1379, 768, 1000), (200, 130, 514), (17, 16, 19), (300, 768, 33),
                                   (16, 16, 15)])
def test_layer_gradients_in_one_launch(fxp, M, K, N):
    say("layer gradients", (M, K, N))
    rng = np.random.default_rng(M + K + N)
    X, W, dY = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (K, N), (M, N)))
    buf = fxp.LayerBuffers(M, K, N)
    Y = fxp.linear_fwd(dev(X), dev(W), buf, seed=2, step=3)
    dX, dW = fxp.linear_bwd(dev(dY), buf, seed=2, step=3)
    Yo, saved = oracle.linear_fwd(X, W, seed=2, step=3)
    dXo, dWo, _ = oracle.linear_bwd(dY, saved, seed=2, step=3)
    assert same_bits(host(Y), Yo) and same_bits(host(dX), dXo) and same_bits(host(dW), dWo)


@pytest.mark.parametrize("batch,M,K,N,transB", [(96, 197, 64, 197, True), (3, 50, 33, 70, False), (7, 65, 80, 97, True), (2, 16, 16, 16, False)])
def test_bmm_gradients_in_one_launch(fxp, batch, M, K, N, transB):
    say("bmm gradients", (batch, M, K, N, transB))
    rng = np.random.default_rng(batch + M + K + N)
    A, dY = rng.standard_normal((batch, M, K)).astype(np.float32), rng.standard_normal((batch, M, N)).astype(np.float32)
    B = rng.standard_normal((batch, N, K) if transB else (batch, K, N)).astype(np.float32)
    buf = fxp.BmmBuffers(batch, M, K, N, transB=transB)
    Y = fxp.bmm_fwd(dev(A), dev(B), buf, seed=2, step=3)
    dA, dB = fxp.bmm_bwd(dev(dY), buf, seed=2, step=3)
    Yo, saved = oracle.bmm_fwd(A, B, transB=transB, seed=2, step=3)
    dAo, dBo, _ = oracle.bmm_bwd(dY, saved, seed=2, step=3)
    assert same_bits(host(Y), Yo) and same_bits(host(dA), dAo) and same_bits(host(dB), dBo)


# a whole number of workgroups, one element and one quad more and less, in one, two and four passes; both sides of the
# size beyond which tensors of long rows are tiled
@pytest.mark.parametrize("rows,cols", [(1, 4096), (1, 4097), (1, 4095), (4, 1025), (1, 4100), (1024, 8192), (1024 * 8192 + 3, 1), (4096, 4096),
                                       (16777213, 1), (65535, 1024), (65536, 1024), (65536, 1020)])
def test_map_row_major_alone(fxp, rows, cols):
    """The row-major copy alone is the one that is written beside a transposed copy."""
    say("map, row-major alone", (rows, cols))
    x = torch.randn((rows, cols), device="cuda")
    x[rows // 2, cols // 3] = float("inf")
    x[rows - 1, cols - 1] = 7.9999999
    e = torch.full((1,), 129, dtype=torch.int32, device="cuda")
    q, qT, alone = (torch.zeros(rows * cols, dtype=torch.int8, device="cuda") for _ in range(3))
    for out, outT in ((q, qT.data_ptr()), (alone, None)):
        assert fxp.lib().fxp_map(x.data_ptr(), rows, cols, e.data_ptr(), out.data_ptr(), outT, 5, 77, 0, 8, None) == 0
    torch.cuda.synchronize()
    assert torch.equal(q, alone)
    n = min(rows * cols, 200000)
    want = oracle.map(host(x).reshape(1, -1)[:, :n], 129, seed=5, stream_id=77)
    assert np.array_equal(host(alone)[:n], want[0])


# contractions of one K step in many small matrices, aligned and ragged: below 16 terms, 16, up to one 64-byte step and a
# byte beyond it; every tile (64 and 128 columns and rows), one matrix per tile and several
@pytest.mark.parametrize("batch,M,N,K", [(600, 16, 16, 16), (513, 33, 40, 15), (700, 17, 70, 64), (600, 70, 17, 63), (520, 130, 129, 48),
                                         (600, 16, 16, 65), (512, 130, 70, 13), (530, 40, 30, 33)])
def test_gemm_batched_one_step(fxp, batch, M, N, K):
    say("batched gemm of one step", (batch, M, N, K))
    rng = np.random.default_rng(batch + M + K)
    A, B = rand_i8(rng, (batch, M, K)), rand_i8(rng, (batch, N, K))
    want = oracle.gemm_batched(A, B, transB=True)
    assert np.array_equal(host(fxp.gemm_batched(dev(A), dev(B))), want)
    e = dev(np.array([121, 130], np.int32))
    assert same_bits(host(fxp.gemm_batched(dev(A), dev(B), e[0:1], e[1:2])).reshape(-1), oracle.unmap(want.reshape(-1), 121, 130))
