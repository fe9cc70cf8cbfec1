"""When the lane kernel is chosen, and its image (no GPU; the host code with the address and
undefined-behaviour sanitizers)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("lane") / "lane_rule")
    subprocess.run(["g++", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-g", "-O2",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "lane_rule.cpp"),
                    os.path.join(ROOT, "paper_2511_17245_amd", "csrc", "sa_host.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("which", ["choice", "image", "levels"])
def test_lane(checker, which):
    out = subprocess.run([checker, which], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stderr[-4000:]
