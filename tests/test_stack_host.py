"""The layer stack's bookkeeping after a copy that HIP refuses (csrc/stack.hip): nothing of the failed step may be taken
for granted by the next ones.  Host code only, against a HIP of plain host memory (stack_host.cpp)."""
import os
import subprocess

from paper_2512_17073_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_steps_after_a_refused_copy(tmp_path):
    objs = []
    for src in (os.path.join(HERE, "stack_host.cpp"), os.path.join(build.CSRC, "stack.hip")):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run([build._hipcc(), "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-x", "hip", "-c", src, "-o", obj], check=True)
        objs.append(obj)
    exe = str(tmp_path / "stack_host")
    subprocess.run(["g++", *objs, "-o", exe], check=True)       # (no HIP runtime: the fake one is in the program)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
