"""A fragment that the orbital-energy gap check rejects costs no product: the
check runs before the first (ia|jb) product (a small one's runs beside it), every
kernel after it does nothing, and the outputs stay unwritten."""
import pytest
import torch

import paper_2410_21888_amd as rm
from gpu_util import say

pytestmark = pytest.mark.gpu


def _run(shape, gap, opts, density):
    nocc, nvir, naux = shape
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    B = 0.1 * torch.randn(nocc, nvir, naux, **kw)
    eo, ev = -1.0 - torch.rand(nocc, **kw), 0.1 + torch.rand(nvir, **kw)
    if not gap:
        ev[nvir // 2] = eo.max() - 1e-3
    nan = lambda *s: torch.full(s, float("nan"), dtype=torch.float64, device="cuda:0")
    out = [nan(2), nan(*shape)] + ([nan(nocc, nocc), nan(nvir, nvir)] if density else [None, None]) + [nan(nocc, nocc)]
    ws = torch.empty(rm.workspace_size(*shape, density=density, opts=opts), dtype=torch.uint8, device="cuda:0")
    rm.timing_enable(True)
    rm.fragment_into(B, eo, ev, *out, workspace=ws, opts=opts)
    stats = {s["name"]: s for s in rm.timing_collect()}
    rm.timing_enable(False)
    return rm.read_status(ws), [t for t in out if t is not None], stats


@pytest.mark.parametrize("density", [True, False])
@pytest.mark.parametrize("shape,group,small", [((5, 25, 90), 0, True), ((20, 100, 400), 0, True),
                                               ((40, 200, 720), 0, False), ((40, 200, 720), 13, False)])
def test_rejected_fragment(shape, group, small, density):
    opts = rm.make_opts(slab_group=group)
    _run(shape, True, opts, density)                      # first call: code load
    st, out, ok = _run(shape, True, opts, density)
    assert st == rm.RIMP2_OK and all(torch.isfinite(t).all() for t in out)
    st, out, bad = _run(shape, False, opts, density)
    assert st == rm.RIMP2_EGAP and all(torch.isnan(t).all() for t in out)
    say("%s group %d density %s: (ia|jb) %.3f ms accepted, %.3f rejected" %
        (shape, group, density, ok["ints_gemm"]["total_ms"], bad["ints_gemm"]["total_ms"]))
    assert ("gap_check" in bad) == (not small)
    if not small:                                         # 0.2 ms or more of product against empty launches
        assert bad["ints_gemm"]["total_ms"] < 0.5 * ok["ints_gemm"]["total_ms"]
