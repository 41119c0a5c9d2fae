"""The plan of rimp2_fragment_noalloc, on the host: a program of the library's
host code alone (no device code, no GPU) prints the slab group and the split
lengths it would run.

Near the size at which the fixed scratch array is full, slabs and split-K
partial sums share it.  The sums that one workgroup runs through serially have to
stay short there (P_ij and P_ab at most 4096 terms: twice the 2048 that the
longest split had where splits only filled the chip), and where there is room for
several orbitals a group the partial sums must not take it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_21888_amd import build as B

PROGRAM = """
#include "%s"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int64_t o = atoi(argv[i]), v = atoi(argv[i + 1]);
    Plan P{};
    const int rc = noalloc_plan(o, v, atoi(argv[i + 2]), atoi(argv[i + 3]), nullptr, &P);
    printf("%%d %%lld %%lld %%lld %%zu\\n", rc, (long long)P.g, (long long)cdiv(P.g * v * v, P.c_ij.splits + !P.density),
           (long long)cdiv(P.g * o * v, P.c_ab.splits + !P.density), P.total);
  }
}
"""
# (nocc, nvir, naux): orbitals a group at least
SIZES = {(51, 427, 1404): 1, (61, 409, 945): 1, (55, 440, 990): 1, (56, 448, 1008): 1, (73, 365, 1314): 1,
         (79, 395, 1422): 1, (30, 150, 540): 20, (39, 212, 746): 6, (61, 305, 1098): 1, (20, 100, 400): 20}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    hipcc = B.hipcc()
    nm = shutil.which("nm") or os.path.join(os.path.dirname(hipcc), "..", "llvm", "bin", "llvm-nm")
    if not os.path.exists(hipcc) or not os.path.exists(nm):
        pytest.skip("no HIP toolchain")
    d = str(tmp_path_factory.mktemp("plan"))
    src, obj, exe = (os.path.join(d, n) for n in ("plan.hip", "plan.o", "plan"))
    with open(src, "w") as f:
        f.write(PROGRAM % os.path.join(B.CSRC, "rimp2.hip"))
    run = lambda *cmd: subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=300).stdout
    run(hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-c", src, "-o", obj)
    image = re.search(r"U (__hip_fatbin\w*)", run(nm, obj)).group(1)   # the device code that is not there
    run(hipcc, obj, "-Wl,--defsym=%s=0" % image, "-o", exe)
    out = {}
    for want in (3, 1):
        lines = run(exe, *[str(a) for s in SIZES for a in (*s, want)]).splitlines()
        out[want] = {s: [int(a) for a in l.split()] for s, l in zip(SIZES, lines)}
    return out


@pytest.mark.parametrize("size", sorted(SIZES))
def test_room_and_serial_sums(plans, size):
    rc, group, pij, pab, total = plans[3][size]
    print(size, "group", group, "P_ij", pij, "P_ab", pab, "MiB", total / 2.0 ** 20)
    assert rc == 0 and total <= 256 << 20
    assert group >= SIZES[size]
    assert pij <= 4096 and pab <= 4096


@pytest.mark.parametrize("size", sorted(SIZES))
def test_gamma_alone_fits(plans, size):
    rc, _, _, _, total = plans[1][size]
    assert rc == 0 and total <= 256 << 20
