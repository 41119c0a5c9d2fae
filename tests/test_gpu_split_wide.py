"""Split Gamma products large enough for the 128 x 128 tile (256 tiles or
more), alone and in a batch, against the FP64 path's Gamma.

Ragged last tiles in both directions, reductions of one and of several
windows, and every digit count that has the wide tile.  Bar: a digit
truncation of 2^-7S relative to the operands' row maxima, times 256 for row
maxima above the typical element and the sum over the reduction, as a relative
Frobenius norm; a wrong digit, row or column is off by 2^-14 or more."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu


def _inputs(nocc, nvir, naux):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(nocc + nvir + naux)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    return (0.3 * torch.randn(nocc, nvir, naux, **kw), -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw))


@pytest.mark.parametrize("shape", [(17, 131, 1990), (40, 230, 520)])
@pytest.mark.parametrize("digits", [3, 4, 5])
def test_wide_gamma(shape, digits):
    B, eo, ev = _inputs(*shape)
    ref = rm.fragment(B, eo, ev, density=False).Gamma
    opts = rm.make_opts(precision=rm.SPLIT_INT8, split_slices_gamma=digits)
    say("wide split Gamma %s digits=%d" % (shape, digits))
    one = rm.fragment(B, eo, ev, density=False, opts=opts).Gamma
    d = dict(B=B, eps_occ=eo, eps_vir=ev, E=torch.zeros(2, dtype=torch.float64, device=B.device),
             Gamma=torch.empty_like(B))
    rm.fragment_batch([d], opts=opts)
    bar = 256.0 * 2.0 ** (-7 * digits)
    for name, got in (("alone", one), ("batch", d["Gamma"])):
        err = float((got - ref).norm() / ref.norm())
        say("  %s: %.2e (bar %.2e)" % (name, err, bar))
        assert err <= bar, (name, err)
