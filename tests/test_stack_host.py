"""Host code of csrc/ that needs no device, compiled into small programs of its own: the layer stack's bookkeeping after a
copy that HIP refuses (stack_host.cpp, against a HIP of plain host memory: nothing of a failed step may be taken for granted by the
next ones), the shares of the decode launches' blocks (plan_host.cpp), and the cut of the offline half's products with the room they
take (gemm_cut_host.cpp)."""
import os
import subprocess

from paper_2512_17073_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def _run(tmp_path, *sources):
    objs = []
    for src in sources:
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run([build._hipcc(), "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-x", "hip", "-c", src, "-o", obj], check=True)
        objs.append(obj)
    exe = str(tmp_path / "program")
    subprocess.run(["g++", *objs, "-o", exe], check=True)       # (no HIP runtime: a fake one is in the program that needs it)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_steps_after_a_refused_copy(tmp_path):
    _run(tmp_path, os.path.join(HERE, "stack_host.cpp"), os.path.join(build.CSRC, "stack.hip"))


def test_shares_of_the_decode_blocks(tmp_path):
    _run(tmp_path, os.path.join(HERE, "plan_host.cpp"))


def test_cut_of_the_fp64_products(tmp_path):
    _run(tmp_path, os.path.join(HERE, "gemm_cut_host.cpp"))
