"""What rimp2_workspace_size asks for beside the slabs (host only).

The split-K partial sums of Gamma, P_ab and P_ij take at most an eighth of the
slab budget each, or 2 GiB; the rest beside the two slabs (pair energies, their
partial sums, alignment) is small.  A Gamma too large for one launch's reduction
is computed without splits, not refused."""
import pytest

import paper_2410_21888_amd as rm

GIB = 1 << 30


@pytest.mark.parametrize("budget", [0, 8 * GIB, 512 << 20])
@pytest.mark.parametrize("size", [(279, 5366, 7205), (196, 1462, 7275), (200, 1800, 6000), (40, 900, 3000),
                                  (9, 8000, 30000), (20, 100, 400)])
def test_partial_sums_are_bounded(size, budget):
    nocc, nvir, naux = size
    opts = rm.make_opts(slab_budget_bytes=budget)
    cap = max((budget or 64 * GIB) // 8, 2 * GIB)
    slab_per_orbital = 16 * nocc * nvir * nvir
    slabs = max(budget or 64 * GIB, slab_per_orbital)
    rest = 8 * nocc * nocc + 16 * (6144 * 2 + nocc * nocc) + (1 << 20)   # pair energies and their partial sums
    for density, products in ((True, 3), (False, 1)):
        total = rm.workspace_size(nocc, nvir, naux, True, density, opts)
        print(size, budget, density, total / GIB)
        assert total <= slabs + products * cap + rest


def test_large_gamma_runs_without_splits():
    # 2^32 elements and a reduction of 33000: no splits for one launch to sum
    total = rm.workspace_size(20, 1650, 131072, True, True)
    assert total <= 16 * (20 * 1650) ** 2 + 2 * 8 * GIB + (1 << 28)
