"""The plan of rimp2_fragment_noalloc, on the host: a program of the library's
host code alone prints the slab group and the split lengths it would run.

Near the size at which the fixed scratch array is full, slabs and split-K
partial sums share it.  The sums that one workgroup runs through serially have to
stay short there (P_ij and P_ab at most 4096 terms: twice the 2048 that the
longest split had where splits only filled the chip), and where there is room for
several orbitals a group the partial sums must not take it."""
import pytest

import host_program

PROGRAM = r"""
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int64_t o = atoi(argv[i]), v = atoi(argv[i + 1]);
    Plan P{};
    const int rc = noalloc_plan(o, v, atoi(argv[i + 2]), atoi(argv[i + 3]), nullptr, &P);
    printf("%d %lld %lld %lld %zu\n", rc, (long long)P.g, (long long)cdiv(P.g * v * v, P.c_ij.splits + !P.density),
           (long long)cdiv(P.g * o * v, P.c_ab.splits + !P.density), P.total);
  }
}
"""
# (nocc, nvir, naux): orbitals a group at least
SIZES = {(51, 427, 1404): 1, (61, 409, 945): 1, (55, 440, 990): 1, (56, 448, 1008): 1, (73, 365, 1314): 1,
         (79, 395, 1422): 1, (30, 150, 540): 20, (39, 212, 746): 6, (61, 305, 1098): 1, (20, 100, 400): 20}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = host_program.build(PROGRAM, str(tmp_path_factory.mktemp("plan")))
    out = {}
    for want in (3, 1):
        lines = host_program.run(exe, *[a for s in SIZES for a in (*s, want)]).splitlines()
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
