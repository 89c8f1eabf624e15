"""How products are cut into slices and sums of slices among lanes (csrc/fxp_gemm_plan.h), on the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2207_08822_amd", "csrc")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    cxx = shutil.which("g++")
    assert cxx, "g++ is part of the image"
    exe = str(tmp_path_factory.mktemp("plan") / "gemm_plan")
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "helpers", "gemm_plan.cpp"), "-o", exe], check=True)

    def run(lines):
        out = subprocess.run([exe], input="".join(" ".join(map(str, l)) + "\n" for l in lines), capture_output=True, text=True, check=True).stdout
        return [list(map(int, l.split())) for l in out.splitlines()]
    return run


@pytest.mark.parametrize("pieces", [1, 1024, 2352, 4096, 16384, 65535, 65536, 1 << 20])
def test_a_lane_of_a_shared_piece_has_a_round_of_slices(ask, pieces):
    splits = list(range(1, 600))
    lanes = [l[0] for l in ask([("reduce", pieces, s, 0) for s in splits])]
    for s, l in zip(splits, lanes):
        assert l in (1, 2, 4, 8, 16, 32), (pieces, s, l)
        assert l == 1 or s // l >= 8, (pieces, s, l)               # eight loads in flight, all of them slices
        assert l == 1 or pieces * l // 2 < 65536, (pieces, s, l)   # and only while half as many lanes leave CUs idle
    assert lanes == sorted(lanes) and (lanes[255] == 32 or pieces * 16 >= 65536)


def test_tiles_of_products(ask):
    """Small tiles where they leave CUs with one each; near two each, not off the 64-byte grid or along very long contractions,
    nor many of a short one that publish their largest magnitude."""
    want = {(1024, 1024, 1024): 1, (1024, 2048, 1024): 1, (1024, 2048, 1984): 1, (1024, 2048, 2000): 0, (2048, 1024, 1776): 0, (1000, 2000, 2032): 0,
            (1024, 1920, 2000): 0, (1024, 1792, 2000): 1, (1024, 2048, 1040): 1, (1300, 1400, 2000): 1, (128, 16384, 2000): 1, (16384, 100, 2032): 1,
            (128, 16384, 4096): 1, (128, 16384, 5120): 0, (64, 16384, 8192): 1, (100, 16384, 12288): 0, (2048, 2048, 1024): 0, (129, 16384, 512): 0}
    assert [g[0] for g in ask([("tiles",) + c for c in want])] == list(want.values())
    short = {(14848, 128, 128): [1, 0], (256, 7232, 256): [1, 0], (9088, 128, 256): [1, 1], (256, 7232, 768): [1, 1], (2048, 2048, 256): [0, 0]}
    assert ask([("tiles",) + c for c in short]) == list(short.values())


SIZES = [1, 16, 49, 784, 6272, 25088, 100352, 133144, 133145, 200704, 802816, 1 << 22]


@pytest.mark.parametrize("Cout", [16, 64, 80, 128, 512, 1024])
def test_weight_gradient_cuts(ask, Cout):
    """Every pixel in one slice, none longer than an int32 sum holds, slices within their workspace; the chip full where there are
    pixels enough for it; many slices only where they are no more bytes than stored patches."""
    cases = [(M, Cout, K) for M in SIZES for K in (16, 64, 144, 576, 1152, 4608)]
    for (M, _, K), (pairs, bm, tiles, slices, per, ws) in zip(cases, ask([("wgrad",) + c for c in cases])):
        where = (M, Cout, K, pairs, bm, tiles, slices, per, ws)
        assert bm == (64 if Cout <= 64 else 128) and tiles == -(-Cout // bm) * -(-K // 128) and not (pairs and bm == 64), where
        assert per % 128 == 0 and (slices - 1) * per < M <= slices * per, where
        assert per <= 133120 or M <= 133144, where
        assert ws == (4 * slices * Cout * K if slices > 1 else 0), where
        assert slices <= 64 or ws <= M * K, where
        most = min(M // 512, max(64, min(512, M // (4 * Cout))))
        assert tiles * slices >= 100 or slices * 1.5 >= min(most, 128 / tiles), where


def test_one_tap_layers_of_few_pixels(ask):
    """1x1 layers whose weight gradient one round of loads of the direct product beats a slice of five to eight stages."""
    want = {(784, 400, 272): 1, (784, 32, 16): 1, (960, 32, 64): 1, (1024, 1024, 16): 1, (576, 256, 128): 1, (512, 256, 128): 0, (576, 64, 256): 0,
            (640, 64, 64): 0, (656, 64, 64): 1, (1040, 128, 128): 0, (784, 800, 384): 0, (980, 256, 64): 1, (980, 256, 272): 1, (940, 256, 272): 0, (980, 64, 64): 0,
            (756, 256, 64): 0, (588, 128, 32): 1, (980, 128, 512): 1, (900, 400, 512): 0, (961, 512, 256): 0, (961, 480, 16): 1, (675, 480, 16): 0,
            (392, 192, 16): 0}
    assert [g[0] for g in ask([("patches",) + c for c in want])] == list(want.values())


def test_weight_gradient_cuts_of_the_gpu_tests(ask):
    """What the shapes of tests/test_gpu_conv_wgrad.py are there for: (pairs, slices, steps of a slice)."""
    cases = {(784, 1024, 4608): (1, 1, 7), (12544, 512, 2304): (1, 7, 14), (560, 1040, 4752): (1, 1, 5), (200704, 16, 16): (0, 224, 7),
             (99910, 32, 16): (0, 157, 5)}
    for got, (case, want) in zip(ask([("wgrad",) + c for c in cases]), cases.items()):
        assert (got[0], got[3], got[4] // 128) == want, (case, got)
