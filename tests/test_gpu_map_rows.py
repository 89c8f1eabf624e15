"""GPU parity of the map's tiles of quads: rows that are not whole quads, bases off the 16-byte grid, tensors whose scale is found
in the same launch - against the CPU oracle, byte for byte."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def fxp():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: there is no CPU path in libfxp")
    from paper_2207_08822_amd import fxp as binding
    binding.lib()
    return binding


def tensor(rows, cols, special):
    rng = np.random.default_rng(rows * 7 + cols)
    x = (rng.standard_normal((rows, cols)) * 3e-3).astype(np.float32)
    if special:
        x.flat[rng.integers(0, x.size, 5)] = np.array([np.inf, -np.inf, np.nan, 1e30, 1e-42], np.float32)
        x.flat[x.size - 1] = -1.9999999
    return x


# windows of a quad and of its parts, a last window that begins in the tensor's short last quad (1154 = 36 x 32 + 2, 3 x 1025),
# one to eight row blocks of a window side by side and more of them, remainders of 1, 2, 3 elements, tiles of 64 and of 128 rows (the
# last five)
SHAPES = [(1, 16), (1, 17), (3, 19), (1, 1154), (3, 1025), (31, 130), (33, 127), (64, 129), (65, 257), (127, 66), (95, 33), (129, 99),
          (250, 99), (5000, 51), (12001, 197), (25200, 149), (33000, 35), (70001, 17),
          (12608, 1001)]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("offset,rounding", [(0, 0), (1, 0), (3, 1)])
def test_map_tiles_of_quads(fxp, rows, cols, offset, rounding):
    say("tiles of quads", (rows, cols), "offset", offset, "rounding", rounding)
    x = tensor(rows, cols, True)
    n, e = rows * cols, 122
    want = oracle.map(x, e, seed=9, stream_id=(3 << 8) | 1, rounding=rounding)
    xd = torch.zeros(n + offset, device="cuda")
    xd[offset:] = dev(x).flatten()
    q, qT = (torch.full((n + 2 * offset + 16,), 77, dtype=torch.int8, device="cuda") for _ in range(2))
    ed = dev(np.array([e], np.int32))
    assert fxp.lib().fxp_map(xd.data_ptr() + 4 * offset, rows, cols, ed.data_ptr(), q.data_ptr() + offset, qT.data_ptr() + 2 * offset, 9,
                             (3 << 8) | 1, rounding, 8, None) == 0
    torch.cuda.synchronize()
    q, qT = host(q), host(qT)
    assert np.array_equal(q[offset:offset + n].reshape(rows, cols), want)
    assert np.array_equal(qT[2 * offset:2 * offset + n].reshape(cols, rows), want.T)
    for a, at in ((q, offset), (qT, 2 * offset)):                      # nothing beyond either copy is touched
        assert (a[:at] == 77).all() and (a[at + n:] == 77).all()


# 114688 elements and one more, one round of eight loads (16384) and beyond, sixteen and eight (49152) and beyond, the narrowest rows
# and narrower ones, one row
@pytest.mark.parametrize("rows,cols", [(256, 256), (7168, 16), (1, 114688), (1, 16), (2, 15), (255, 257), (448, 257), (1, 114689), (1, 1154), (128, 128), (129, 127), (192, 256), (4, 12289), (9, 12288),
                                       (200, 100), (33, 31)])
@pytest.mark.parametrize("kind", ["plain", "special", "zero"])
def test_scale_and_map_of_small_tensors(fxp, rows, cols, kind):
    say("small scale + map", (rows, cols), kind)
    x = tensor(rows, cols, kind == "special") * np.float32(0.0 if kind == "zero" else 1.0)
    x[np.isnan(x)] = 0.0 if kind == "zero" else np.nan
    x.flat[0 if cols % 2 else x.size - 1] *= 64.0                      # the largest at one of the ends
    for offset in (0, 1):
        xd = torch.zeros(x.size + offset, device="cuda")
        xd[offset:] = dev(x).flatten()
        e, q, qT = fxp.scale_map(xd[offset:].view(rows, cols), seed=4, stream_id=9, want_qT=True)
        e_want = oracle.scale(x)
        assert int(e[0]) == e_want
        want = oracle.map(x, e_want, seed=4, stream_id=9)
        assert np.array_equal(host(q), want) and np.array_equal(host(qT), want.T)


@pytest.mark.parametrize("a,b", [((256, 256), (256, 128)), ((197, 64), (64, 80)), ((100, 50), (300, 300)), ((2364, 197), (2364, 64)),
                                 ((500, 70), (70, 512)), ((64, 200), (200, 333))])
def test_two_tensors_of_a_launch(fxp, a, b):
    """Both small, one of them small, tiles of quads beside an aligned tensor of another tile width."""
    say("scale + map of two", a, b)
    xa, xb = tensor(*a, False), tensor(*b, False) * np.float32(50.0)
    e, (qa, qaT), (qb, qbT) = fxp.scale_map2(dev(xa), dev(xb), seed=11, stream_ids=(512, 513))
    for x, ee, q, qT, sid in ((xa, e[0], qa, qaT, 512), (xb, e[1], qb, qbT, 513)):
        assert int(ee) == oracle.scale(x)
        want = oracle.map(x, int(ee), seed=11, stream_id=sid)
        assert np.array_equal(host(q), want) and np.array_equal(host(qT), want.T)
