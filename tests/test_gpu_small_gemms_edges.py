"""The one launch of Gamma, P_ab and P_ij at the edges of what the plan gives to
it, each shape asserted to take it: the smallest runs, an odd naux just past one
tile, and for few, middling and many occupied orbitals the largest nvir or naux
with tiles of 64/64/32, with even and odd runs.  And shapes just outside, asserted
to take separate launches.  Bit for bit against the general loader's separate
launches, which sum every element in the same order."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu

ONE_LAUNCH = [(1, 16, 2), (2, 16, 65), (3, 17, 67), (5, 25, 90), (20, 100, 399), (12, 256, 1801), (31, 245, 1801),
              (48, 63, 129), (64, 61, 1801)]
SEPARATE = [(2, 17, 9),       # an odd naux narrower than a tile
            (31, 65, 130),    # P_ab in tiles of 96
            (33, 66, 96)]     # P_ij in tiles of 64


@pytest.mark.parametrize("shape", ONE_LAUNCH + SEPARATE)
def test_edges(shape):
    nocc, nvir, naux = shape
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(nocc * nvir + naux)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    B = 0.3 * torch.randn(nocc, nvir, naux, **kw)
    eo, ev = -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw)
    rm.timing_enable(True)
    one = rm.fragment(B, eo, ev)
    roles = {r["name"] for r in rm.timing_collect()}
    rm.timing_enable(False)
    say("small GEMMs %s: %s" % (shape, sorted(roles)))
    separate = {"gamma_gemm", "pab_gemm", "pij_gemm"}
    if shape in ONE_LAUNCH:
        assert "small_gemms" in roles and not roles & separate
    else:
        assert "small_gemms" not in roles and roles >= separate
    apart = rm.fragment(B, eo, ev, opts=rm.make_opts(gemm_loader=1))
    for name, a, b in zip(one._fields, one, apart):
        assert torch.isfinite(a).all() and torch.equal(a, b), name
