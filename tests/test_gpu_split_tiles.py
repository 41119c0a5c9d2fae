"""Split products in the 128 x 128 tile against the same digit products in the
64 x 64 tile, bit for bit: the digit sums are exact integers, and both tiles
combine and scale them alike, so any lost, doubled or misplaced digit, row or
column shows, in the last ragged tiles too.

Which tile a product takes depends on how many tiles of 128 there are (256 or
more: 128 x 128), over a batch's wave together: the same fragment takes the small
one alone and the large one beside a copy of itself, or the large one in one slab
and the small one in several.  Sizes with ragged last tiles in both directions and
reductions of one and of several windows, every digit count with the wide tile."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu


def _inputs(nocc, nvir, naux):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(nocc + nvir + naux)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    return 0.3 * torch.randn(nocc, nvir, naux, **kw), -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw)


def _wide(rows, cols):
    t = {s: -(-rows // s) * (-(-cols // s)) for s in (64, 128)}
    return t[128], 4 * t[128] < 1.2 * t[64]


def _batch(d, copies, opts):
    frags = [dict(B=d[0], eps_occ=d[1], eps_vir=d[2], E=torch.zeros(2, dtype=torch.float64, device="cuda:0"),
                  Gamma=torch.full_like(d[0], float("nan"))) for _ in range(copies)]
    rm.fragment_batch(frags, opts=opts)
    torch.cuda.synchronize()
    return [f["Gamma"] for f in frags]


@pytest.mark.parametrize("digits", [3, 4, 5])
@pytest.mark.parametrize("shape", [(17, 131, 1000), (40, 230, 380)])
def test_grouped_gamma(shape, digits):
    tiles, pays = _wide(shape[0] * shape[1], shape[2])
    assert pays and tiles < 256 <= 2 * tiles
    d = _inputs(*shape)
    opts = rm.make_opts(precision=rm.SPLIT_INT8, split_slices_gamma=digits)
    say("grouped Gamma %s digits %d" % (shape, digits))
    small, = _batch(d, 1, opts)
    assert torch.isfinite(small).all()
    for wide in _batch(d, 2, opts):
        assert torch.equal(small, wide)


@pytest.mark.parametrize("digits", [3, 4, 5])
@pytest.mark.parametrize("shape,group", [((17, 131, 1990), 5), ((40, 230, 520), 13)])
def test_gamma_of_one_slab_and_of_several(shape, group, digits):
    tiles, pays = _wide(shape[0] * shape[1], shape[2])
    assert pays and tiles >= 256 > _wide(group * shape[1], shape[2])[0]
    d = _inputs(*shape)
    out = []
    for g in (0, group):
        say("Gamma %s digits %d slab_group %d" % (shape, digits, g))
        out.append(rm.fragment(*d, opts=rm.make_opts(precision=rm.SPLIT_INT8, split_slices_gamma=digits, slab_group=g)))
    assert torch.isfinite(out[0].Gamma).all()
    assert torch.equal(out[0].Gamma, out[1].Gamma)


@pytest.mark.parametrize("digits", [3, 4, 5])
def test_integrals(digits):
    """(ia|jb): a batch's products always take the small tile, a fragment's own
    the wide one at these digit counts; Gamma carries every integral."""
    shape = (17, 131, 1990)
    tiles, pays = _wide(shape[0] * shape[1], shape[0] * shape[1])
    assert pays and tiles >= 256
    d = _inputs(*shape)
    opts = rm.make_opts(precision=rm.SPLIT_INT8, split_slices=digits)
    say("(ia|jb) %s digits %d" % (shape, digits))
    wide = rm.fragment(*d, opts=opts).Gamma
    small, = _batch(d, 1, opts)
    assert torch.isfinite(wide).all() and torch.equal(wide, small)
