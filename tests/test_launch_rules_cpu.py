"""The rules of csrc/launch_rules.h, compiled for the host with g++ and checked
without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_04894_amd", "csrc")


def run(tmp_path, body):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "launch_rules.h"\nusing namespace fmm::rules;\nint main() {\n' + body + "}\n")
    subprocess.run([gxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()


@pytest.mark.parametrize("nseg,entries,f32,waves", [
    # entries enough for all waves: by the number of segments
    (1, 8, 0, 8), (512, 512 * 30, 0, 8), (513, 513 * 30, 0, 4), (2048, 2048 * 4, 0, 4), (2049, 2049 * 30, 0, 1),
    # binary64: no more waves than the segments have work for
    (64, 64 * 4, 0, 8), (64, 64 * 4 - 1, 0, 4), (64, 64 * 2, 0, 4), (64, 64 * 2 - 1, 0, 1), (64, 64, 0, 1),
    (1500, 1500 * 2, 0, 4), (1500, 1500, 0, 1), (1, 1, 0, 1),
    # binary32 deals out chunks, not entries
    (64, 64, 1, 8), (1500, 1500, 1, 4), (4000, 4000, 1, 1),
])
def test_near_field_waves(tmp_path, nseg, entries, f32, waves):
    assert run(tmp_path, f'std::printf("%d\\n", p2p_waves({nseg}, {entries}, {f32}));\n') == [str(waves)]


@pytest.mark.parametrize("nseg,smallest,largest,chunked", [
    # the largest segment decides, down to 8,192 points in the smallest
    (1, 32_768, 32_768, 1), (1, 32_767, 32_767, 0), (2, 20_000, 4_000_000, 1), (4, 8_192, 32_768, 1),
    (4, 8_191, 4_000_000, 0), (4, 9_000, 32_767, 0), (512, 32_768, 40_000, 1), (1024, 32_768, 40_000, 0),
])
def test_chunked_rounds(tmp_path, nseg, smallest, largest, chunked):
    assert run(tmp_path, f'std::printf("%d\\n", round_chunked({nseg}, {smallest}, {largest}));\n') == [str(chunked)]
