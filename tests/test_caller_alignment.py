"""Callers' buffers are only known to be aligned like one element, so the kernels may not claim
more: the row-wise kernels compiled to LLVM IR for gfx950 (no GPU needed), and the alignment of
every vector store read from it. (The hardware serves such accesses at any alignment of four
bytes; what must not happen is a promise to the compiler that the caller never made.)"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ELEM = {"float": 4, "half": 2, "bfloat": 2}


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    ll = str(tmp_path_factory.mktemp("ir") / "norm_rope.ll")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-x",
                    "hip", "--offload-device-only", "-emit-llvm", "-S", "-o", ll,
                    os.path.join(ROOT, "paper_2606_05981_amd", "csrc", "norm_rope.hip")], check=True,
                   capture_output=True)
    with open(ll) as f:
        text = f.read()
    return {m.group(1): m.group(0) for m in re.finditer(r"^define[^\n]* @(\w+)\(.*?^}", text, re.S | re.M)}


def vector_ops(body, op):
    return [(m.group(1), int(m.group(2)))
            for m in re.finditer(r"%s <\d+ x (\w+)>[^\n]*? ptr addrspace\(1\) [^\n]*?align (\d+)" % op, body)]


def test_residual_add(kernels):
    body = [b for k, b in kernels.items() if "k_resid_add" in k]
    assert len(body) == 1
    stores, loads = vector_ops(body[0], "store"), vector_ops(body[0], "load")
    assert stores == [("float", 4)]                       # h, the caller's stream
    assert loads.count(("float", 4)) == 1                 # h; the partial sums are the library's, 16 bytes
    assert all(a == 16 for t, a in loads if (t, a) != ("float", 4)) and len(loads) > 1


def test_norm_outputs(kernels):
    bodies = [b for k, b in kernels.items() if "k_rmsnorm_vec" in k]
    assert bodies
    n = 0
    for b in bodies:
        for elem, align in vector_ops(b, "store"):        # out and copy_to
            n += 1
            assert align <= ELEM[elem], (elem, align)
    assert n > 0
