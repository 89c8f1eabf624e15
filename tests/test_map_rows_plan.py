"""How tensors are cut into tiles of quads (csrc/fxp_map_plan.h), on the host: every element lies in one window, every quad that a
window meets has a lane, the reciprocal divides exactly, and the addressing stays in 32 bits."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2207_08822_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++")
    assert cxx, "g++ is part of the image"
    exe = str(tmp_path_factory.mktemp("plan") / "map_rows_plan")
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "helpers", "map_rows_plan.cpp"), "-o", exe], check=True)

    def ask(cases):
        out = subprocess.run([exe], input="".join("%d %d %d\n" % c for c in cases), capture_output=True, text=True, check=True).stdout
        return [dict(zip(("tr", "windows", "width", "quads", "blocks", "exact", "scan", "flat"), map(int, l.split()))) for l in out.splitlines()]
    return ask


@pytest.mark.parametrize("rows", [1, 31, 129, 12608, 1 << 20])
def test_every_element_has_one_lane(plan, rows):
    cases = [(rows, c, tr) for c in list(range(4, 300)) + [1000, 1001, 3071, 3072, (1 << 22) - 4, (1 << 22) - 1] for tr in (0, -1, 64, 128)]
    for (_, cols, tr), p in zip(cases, plan(cases)):
        where = (rows, cols, tr, p)
        assert p["exact"] and p["width"] <= (32 if tr < 0 and rows > 16 else 128) and p["tr"] in (32, 64, 128), where
        assert (p["windows"] - 1) * p["width"] < cols <= p["windows"] * p["width"], where
        assert p["blocks"] == -(-rows // p["tr"]) * p["windows"], where
        # the most quads that `width` columns meet: from any element where rows shift, from a quad's first where they do not
        shifts = range(4) if cols % 4 else (0,)
        assert all(p["width"] * w % 4 == 0 for w in range(p["windows"])) or cols % 4, where
        assert p["quads"] >= max(-(-(s + min(p["width"], cols)) // 4) for s in shifts), where
        assert p["tr"] * cols + 128 < 1 << 30, where                  # four-byte offsets of a tile's elements below 2^32


@pytest.mark.parametrize("rows", [40, 64, 1379, 12608, 28800, 1 << 20])
def test_rounds_are_filled(plan, rows):
    """No window meets more quads than the lanes of a round have rows for; where there are tiles for every CU, the chosen height and
    windows leave no more lanes idle than the plainest cut of that height."""
    cols = list(range(16, 400)) + [1000, 1001, 3071, 3072, 50257]
    best, plain = (plan([(rows, c, tr) for c in cols]) for tr in (0, 32))

    def busy(p, c):
        rounds = -(-p["tr"] * p["quads"] // 1024)
        return rows * c / 4 / (rounds * 1024 * (-(-p["blocks"] // 256) * 256))
    for c, p, q in zip(cols, best, plain):
        assert p["quads"] <= 32 and q["quads"] <= 32, (rows, c, p, q)
        assert q["blocks"] < 512 and p == q or p["blocks"] >= 512 and busy(p, c) >= 0.87 ** 2 * busy(q, c), (rows, c, p, q)


def test_heights_of_the_gpu_tests(plan):
    """The heights (and windows) that shapes of tests/test_gpu_map_rows.py are there for."""
    want = {(5000, 51): (32, 1), (12001, 197): (64, 4), (25200, 149): (64, 3), (33000, 35): (128, 2), (70001, 17): (128, 1), (12608, 1001): (128, 11)}
    got = plan([(r, c, 0) for r, c in want])
    assert [(p["tr"], p["windows"]) for p in got] == list(want.values())


def test_small_tensors(plan):
    got = plan([(256, 256, -1), (1, 114688, -1), (7168, 16, -1), (7645, 15, -1), (449, 256, -1), (448, 256, -1), (1, 114689, -1), (0, 16, -1)])
    assert [p["scan"] for p in got] == [1, 0, 1, 0, 0, 1, 0, 0]


def test_scan_of_few_rows(plan):
    """What a CU reads of a tensor whose scale every workgroup finds for itself stays within what one workgroup reads of the largest,
    whatever the shape: few rows are many windows."""
    sizes = [1000, 16384, 32768, 50257, 65536, 98304, 100352, 114688]
    cases = [(r, n // r, -1) for n in sizes for r in (1, 2, 3, 4, 8, 9, 16, 17, 24, 31, 32, 33, 64, 256) if n // r >= 16]
    for (rows, cols, _), p in zip(cases, plan(cases)):
        reads = -(-p["blocks"] // 256) * rows * cols
        assert p["scan"] == (reads <= 112 * 1024), (rows, cols, p)
        assert rows < 8 or p["blocks"] <= 256, (rows, cols, p)          # eight rows and more: never more workgroups than CUs
    shapes = [(1, 114688, -1), (2, 50257, -1), (1, 65536, -1), (4, 25088, -1), (8, 10000, -1), (1, 32768, -1)]
    assert [p["scan"] for p in plan(shapes)] == [0, 0, 0, 1, 1, 1]


@pytest.mark.parametrize("cols", [1, 3, 17, 131])
def test_flat_run_beside_tiles_fills_the_chip(plan, cols):
    """A flat tensor's workgroups in a launch with tiles of quads: 4096 elements for every 32 rows of height, a thousand workgroups if
    the tensor has them, and no smaller than that takes."""
    rows = [10, 1000, 50176, 200704, 401408, 1605632, 10 ** 7]
    for (r, _, _), p in zip([(r, cols, 0) for r in rows], plan([(r, cols, 0) for r in rows])):
        n = r * cols
        blocks = -(-n // (4096 * p["flat"] // 32))
        assert p["flat"] in (32, 64, 128) and blocks >= min(1024, -(-n // 4096)), (r, cols, p, blocks)
        assert p["flat"] == 128 or -(-n // (4096 * p["flat"] // 16)) < 1024, (r, cols, p, blocks)
