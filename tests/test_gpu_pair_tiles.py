"""(ia|jb) launches that hold workgroups for the kept tiles only (pairs j >=
k of a slab group): every kept tile is decoded once, whatever the raster.

Each shape runs the energy with one slab (every pair block from one launch)
and with small slab groups (other launches, other decodes).  An element of
(ia|jb) is the same sum in the same order in both, so e_ij differ by the order
of the amplitude pass's compensated sums alone: 1e-13 relative.  The shapes:
one raster group, a ragged last group, blocks narrower than a tile, and more
than 64 raster groups of 8 tiles of 128 rows (the decode's lanes wrap)."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,g", [((3, 5, 6), 1), ((9, 128, 16), 4), ((13, 211, 18), 5), ((40, 33, 20), 7),
                                     ((82, 808, 2), 20)])
@pytest.mark.parametrize("precision", [rm.FP64, rm.SPLIT_INT8])
def test_one_slab_equals_small_groups(shape, g, precision):
    nocc, nvir, naux = shape
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(nocc + nvir)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    B = 0.3 * torch.randn(nocc, nvir, naux, **kw)
    eo, ev = -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw)
    say("pair tiles nocc=%d nvir=%d naux=%d groups of %d" % (nocc, nvir, naux, g))
    one = rm.fragment(B, eo, ev, gamma=False, density=False, opts=rm.make_opts(precision=precision))
    few = rm.fragment(B, eo, ev, gamma=False, density=False, opts=rm.make_opts(precision=precision, slab_group=g))
    a, b = one.e_pair, few.e_pair
    assert torch.isfinite(a).all()
    assert ((a - b).abs() <= 1e-13 * b.abs()).all()
