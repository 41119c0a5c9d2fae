"""The fast GEMM loader at odd sizes against the general loader, bit for bit
(both sum every element in the same order).

Every operand form that reached the general loader before: odd row strides
(pairs at 8-byte addresses), odd reduction lengths (a ragged last element),
odd numbers of columns or rows of an N- or M-contiguous operand (the last
pair is read one element early: N = 129 and 257 leave one column in the last
tile), odd runs (pairs that lie in two runs), one column, and B at an address
that is not 16-byte aligned."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu

SHAPES = [(1, 17, 1), (1, 2, 3), (2, 17, 15), (3, 17, 33), (3, 19, 129), (5, 33, 257), (3, 129, 31), (7, 65, 47),
          (1, 257, 18), (5, 16, 129), (4, 15, 130)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("density", [True, False])
@pytest.mark.parametrize("shift", [0, 1])
def test_odd_sizes_fast_equals_general(shape, density, shift):
    nocc, nvir, naux = shape
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1000 * nocc + nvir + naux)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    flat = 0.3 * torch.randn(nocc * nvir * naux + 1, **kw)
    B = flat[shift:shift + nocc * nvir * naux].view(nocc, nvir, naux)   # shift 1: B at 8 bytes past a boundary
    eo, ev = -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw)
    for g in sorted({0, 1, max(1, nocc // 2)}):
        say("odd loader %s density=%s shift=%d slab_group=%d" % (shape, density, shift, g))
        fast = rm.fragment(B, eo, ev, density=density, opts=rm.make_opts(slab_group=g))
        general = rm.fragment(B, eo, ev, density=density, opts=rm.make_opts(slab_group=g, gemm_loader=1))
        for name, a, b in zip(fast._fields, fast, general):
            if a is not None:
                assert torch.isfinite(a).all() and torch.equal(a, b), (g, name)
