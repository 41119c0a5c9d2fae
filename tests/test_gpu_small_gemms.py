"""Gamma, P_ab and P_ij of a small fragment in one launch (gemm_f64_tail)
against the separate launches that the general loader takes, bit for bit: both
sum every element in the same order.  Sizes: one tile of each product, several,
odd and even runs (both loader levels), split reductions, and the largest the
plan gives to the one launch's tiles."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 16, 2), (2, 17, 9), (5, 25, 90), (8, 40, 144), (9, 45, 162), (20, 100, 400),
                                   (21, 63, 128), (31, 65, 130), (33, 66, 96)])
def test_one_launch_equals_separate_launches(shape):
    nocc, nvir, naux = shape
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(nocc * nvir + naux)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    B = 0.3 * torch.randn(nocc, nvir, naux, **kw)
    eo, ev = -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw)
    say("small GEMMs %s" % (shape,))
    rm.timing_enable(True)
    one = rm.fragment(B, eo, ev)
    roles = {r["name"] for r in rm.timing_collect()}
    rm.timing_enable(False)
    apart = rm.fragment(B, eo, ev, opts=rm.make_opts(gemm_loader=1))
    for name, a, b in zip(one._fields, one, apart):
        assert torch.isfinite(a).all() and torch.equal(a, b), name
    if shape == (20, 100, 400):
        assert "small_gemms" in roles and "gamma_gemm" not in roles
