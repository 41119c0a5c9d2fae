"""Builds and runs small programs of the library's host code alone (no device
code, no GPU): plans and tables as the library would use them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_21888_amd import build as B


def build(body: str, folder: str) -> str:
    """Path of a program that includes csrc/rimp2.hip and has `body` after it."""
    hipcc = B.hipcc()
    nm = shutil.which("nm") or os.path.join(os.path.dirname(hipcc), "..", "llvm", "bin", "llvm-nm")
    if not os.path.exists(hipcc) or not os.path.exists(nm):
        pytest.skip("no HIP toolchain")
    src, obj, exe = (os.path.join(folder, "program" + e) for e in (".hip", ".o", ""))
    with open(src, "w") as f:
        f.write('#include "%s"\n#include <cstdio>\n#include <cstdlib>\n%s' % (os.path.join(B.CSRC, "rimp2.hip"), body))
    run(hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-c", src, "-o", obj)
    image = re.search(r"U (__hip_fatbin\w*)", run(nm, obj)).group(1)   # the device code that is not there
    run(hipcc, obj, "-Wl,--defsym=%s=0" % image, "-o", exe)
    return exe


def run(*cmd: str) -> str:
    return subprocess.run([str(c) for c in cmd], check=True, capture_output=True, text=True, timeout=300).stdout
