"""A batch's launches that fail half way leave nothing on the side streams that the caller's stream does not wait for
(no GPU: launches, events and waits that are only written down stand before the runtime's)."""
import os
import subprocess

from paper_2511_17245_amd import build as hipbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_side_streams_are_joined(tmp_path):
    if not os.path.exists(hipbuild.LIB):
        hipbuild.build()
    exe = str(tmp_path / "batch_join")
    pkg = os.path.dirname(hipbuild.LIB)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "batch_join.cpp"),
                    "-o", exe, "-L", pkg, "-lsa", f"-Wl,-rpath,{pkg}", "-L/opt/rocm/lib", "-lamdhip64"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
