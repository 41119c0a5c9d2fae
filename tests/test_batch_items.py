"""Work items of a batch's grouped (ia|jb) launch, on the host: one for each tile
that holds a pair j >= k, and none for the others (tiles that only other rows of
their raster group need end at once, and leave CUs idle)."""
import pytest

import host_program

PROGRAM = r"""
int main(int argc, char** argv) {
  for (int i = 1; i + 2 < argc; i += 3) {
    rimp2_frag_desc d{};
    d.nocc = atoi(argv[i]); d.nvir = atoi(argv[i + 1]); d.naux = atoi(argv[i + 2]);
    double* p = (double*)4096;
    d.B = d.eps_occ = d.eps_vir = p; d.E = d.Gamma = d.P_ij = d.P_ab = p;
    rimp2_batch_s B;
    if (batch_plan(1, &d, nullptr, &B)) return 1;
    for (int c = 0; c < 2; ++c)
      printf("%d %lld ", B.waves[0].lists[0][c][0].bm, (long long)B.waves[0].lists[0][c][0].items);
    printf("\n");
  }
}
"""
SIZES = [(1, 7, 9), (5, 25, 90), (20, 100, 400), (21, 103, 371), (40, 200, 720), (61, 305, 1098), (3, 600, 1800)]


@pytest.fixture(scope="module")
def items(tmp_path_factory):
    exe = host_program.build(PROGRAM, str(tmp_path_factory.mktemp("items")))
    lines = host_program.run(exe, *[a for s in SIZES for a in s]).splitlines()
    return {s: [int(a) for a in l.split()] for s, l in zip(SIZES, lines)}


@pytest.mark.parametrize("size", SIZES)
def test_items_are_the_kept_tiles(items, size):
    nocc, nvir, _ = size
    n = nocc * nvir
    for bm, got in (items[size][:2], items[size][2:]):
        tiles = range(-(-n // bm))
        kept = sum((min(n, tn * bm + bm) - 1) // nvir >= tm * bm // nvir for tm in tiles for tn in tiles)
        assert got == kept, (bm, got, kept)
