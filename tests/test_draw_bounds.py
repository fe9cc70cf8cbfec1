"""The heat bath's draws by the inverse of the distribution (csrc/sa_draw.h, compiled for the host) against
113-bit arithmetic and against the weights added one by one: the stated error bounds, the tails, ranges past
65536 values, U = 0, and the margins that pass over a draw (no GPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("draw") / "draw_bounds")
    subprocess.run(["g++", "-std=gnu++17", "-O2", "-ffp-contract=off", "-Wno-unused-function",
                    os.path.join(ROOT, "tests", "draw_bounds.cpp"), "-o", exe, "-lquadmath"], check=True)
    return exe


@pytest.mark.parametrize("which", ["single", "decided", "sums", "margins"])
def test_draws(checker, which):
    out = subprocess.run([checker, which], capture_output=True, text=True, timeout=300)
    print(out.stdout)
    assert out.returncode == 0 and out.stdout.strip().endswith("ok"), out.stdout + out.stderr[-4000:]
