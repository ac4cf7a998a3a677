"""The persistent loops hand words from one workgroup to the next with stores,
a wait for them and a flag.  What the compiler is given must keep that order
by itself: in the device code's LLVM IR every wait stands between two fences
(of one thread: no instructions), which no store may be moved across."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1408_1605_amd", "csrc")


@pytest.mark.parametrize("source", ["smallloop.hip", "msloop.hip"])
def test_waits_are_fenced(source, tmp_path):
    from paper_1408_1605_amd import build
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    ll = str(tmp_path / "k.ll")
    subprocess.run([hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only",
                    "-S", "-emit-llvm", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, source), "-o", ll], check=True, capture_output=True)
    lines = [x.strip() for x in open(ll)]
    waits = [i for i, x in enumerate(lines) if re.search(r"call void @llvm\.amdgcn\.s\.waitcnt\(", x)]
    assert waits
    fence = 'fence syncscope("singlethread") seq_cst'
    for i in waits:
        assert lines[i - 1] == fence and lines[i + 1] == fence, "\n".join(lines[i - 3:i + 3])
