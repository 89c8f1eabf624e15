"""How a map launch cuts a tensor up (csrc/fxp_map_plan.h), on the host: every tensor is covered by the kernel it is given,
whatever asks for the plan - the launch that takes a guessed scale cuts into tiles also what an ordinary map takes flat."""
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
    exe = str(tmp_path_factory.mktemp("plan") / "map_plan")
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "helpers", "map_plan.cpp"), "-o", exe], check=True)

    def ask(*cases):
        text = "".join("%d %d %d %d\n" % c for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [dict(zip(("tc", "passes", "tiles", "any", "flat", "tile_path", "both"), map(int, l.split()))) for l in out.splitlines()]
    return ask


SIZES = [1, 3, 4, 15, 16, 17, 64, 100, 1020, 1024, 1 << 16, (1 << 22) - 4, 1 << 22, (1 << 22) + 1, 1 << 26, (1 << 32) - 1, 1 << 32]


def test_tiles_only_where_their_addressing_reaches(plan):
    cases = [(r, c, a, t) for r in SIZES for c in SIZES for a in (0, 1) for t in (0, 1)]
    for (rows, cols, aligned, transposed), p in zip(cases, plan(*cases)):
        where = (rows, cols, aligned, transposed, p)
        if p["tiles"]:
            # element offsets from a tile's origin and the transposed copy's row count are 32-bit, a launch has fewer than
            # 2^30 tiles, and a short unaligned row is not tiled
            tall = 128 if p["tc"] == 128 else 256
            assert tall * cols + p["tc"] < 1 << 32 and rows < 1 << 32, where
            assert -(-rows // (tall // 4)) * -(-cols // p["tc"]) < 1 << 30, where
            assert p["any"] == (cols % 4 != 0 or not aligned) and (not p["any"] or cols >= 16), where
        assert not (p["flat"] and transposed), where
        assert p["tile_path"] <= (p["tiles"] or p["flat"]), where
    # whether a tensor can be tiled does not depend on the copies that are wanted
    both = {c: p["tiles"] for c, p in zip(cases, plan(*cases))}
    assert all(t == both[c[:3] + (1,)] for c, t in both.items())


@pytest.mark.parametrize("rows,cols", [(4, 1 << 22), (1, 1 << 24), (1 << 32, 16)])
def test_a_flat_tensor_may_be_beyond_tiles(plan, rows, cols):
    """What a caller that cuts into tiles must not take from the flat path: rows of 2^22 columns and 2^32 rows."""
    p, = plan((rows, cols, 1, 0))
    assert p["flat"] and p["tile_path"] and not p["tiles"]


def test_row_major_alone(plan):
    """Flat, but tiles for long rows from 2^26 elements on, unless they are off the grid."""
    got = plan((65535, 1024, 1, 0), (65536, 1024, 1, 0), (65536, 1024, 0, 0), (1 << 20, 1020, 1, 0), (65536, 1025, 1, 0))
    assert [p["flat"] for p in got] == [1, 0, 1, 1, 1]


@pytest.mark.parametrize("image,weights,both", [((25088, 128, 1, 0), (128, 1152, 1, 1), 1), ((50176, 64, 1, 0), (64, 576, 1, 1), 1),
                                                ((200704, 4, 1, 0), (128, 4, 1, 1), 0), ((524288, 4, 1, 0), (128, 36, 1, 1), 0),
                                                ((25088, 128, 0, 0), (128, 1152, 1, 1), 0), ((25088, 48, 1, 0), (96, 432, 1, 1), 0),
                                                ((25088, 56, 1, 0), (64, 576, 1, 1), 1), ((25088, 52, 1, 0), (64, 576, 1, 1), 0),
                                                ((25088, 128, 1, 0), (64, 576, 1, 1), 0), ((25088, 3, 1, 0), (64, 147, 1, 1), 0)])
def test_an_image_and_its_weights(plan, image, weights, both):
    """Tiles for both: one tile width, aligned, and rows that fill the tiles."""
    got = plan(image, weights)
    assert got[0]["flat"] and got[1]["both"] == both
