"""How sums of slices are cut up (csrc/fxp_gemm_plan.h), on the host."""
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
    lanes = [l[0] for l in ask([("reduce", pieces, s) for s in splits])]
    for s, l in zip(splits, lanes):
        assert l in (1, 2, 4, 8, 16, 32), (pieces, s, l)
        assert l == 1 or s // l >= 8, (pieces, s, l)               # eight loads in flight, all of them slices
        assert l == 1 or pieces * l // 2 < 65536, (pieces, s, l)   # and only while half as many lanes leave CUs idle
    assert lanes == sorted(lanes) and (lanes[255] == 32 or pieces * 16 >= 65536)
