"""Ordering of the gradient kernel's partial loss in LDS, read from the code compiled for the GPU:
every lane of a wavefront writes its own value and one lane then reads them all, so a fence has
to stand between, or the compiler may take the reads first."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_14505_amd", "csrc")


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    """name -> body of learned.hip's device functions, in source order (no optimisation passes)."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("lds_order") / "learned.ll")
    subprocess.run([hipcc, "--offload-arch=gfx950", "--cuda-device-only", "-O1", "-std=c++17", "-Xclang",
                    "-disable-llvm-passes", "-emit-llvm", "-S", os.path.join(CSRC, "learned.hip"), "-o", out],
                   check=True, capture_output=True)
    with open(out) as fh:
        text = fh.read()
    return dict(re.findall(r"^define [^@]*@([\w.$]+)\(.*?\{\n(.*?)^\}", text, re.M | re.S))


def test_partial_loss_is_written_before_it_is_read(functions):
    fences = [name for name, body in functions.items() if re.search(r"^\s*fence ", body, re.M)]
    body = next(b for name, b in functions.items() if "grad_kernelEP" in name)
    uses = [m.start() for m in re.finditer(r"@\w*grad_kernel\w*lsum\b", body)]
    assert len(uses) == 2, "one write and one read of the lanes' partial sums"
    between = body[uses[0]:uses[1]]
    assert re.search(r"^\s*fence ", between, re.M) or any(f"@{name}(" in between for name in fences)
