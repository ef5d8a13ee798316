"""The nested-dissection plan cuts large parts on threads of their own; where the
process can have no more threads it cuts them itself, to the same order."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_08594_amd", "csrc")


def test_plan_without_threads(tmp_path):
    exe = str(tmp_path / "nd_threads")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-pthread", f"-I{CSRC}",
                           os.path.join(ROOT, "tests", "native", "nd_threads.cpp"),
                           os.path.join(CSRC, "msp_nd.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout.strip()) == (0, "same"), r.stderr
