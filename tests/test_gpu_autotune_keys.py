"""The autotuner keeps apart what its table cannot name by one candidate list.

Two slab groups give one GEMM shape (M, N, K, split length) different tiles of
the plan: the ragged last group of slab_group = 8 and the full groups of 4 at
nocc = 20, nvir = 100, naux = 1000 share Gamma's, with plan tiles of 128 and 64.
And batches with the fast and with the general loader time different kernels.
Each has an entry of its own, whose first candidate is its plan's tile and whose
launches are all its own; results are bit for bit those of the untuned calls."""
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


def test_one_shape_under_two_plans():
    d = _inputs(20, 100, 1000)
    rm.autotune_reset()
    calls = {8: 6, 4: 3}
    for group, n in calls.items():
        ref = rm.fragment(*d, opts=rm.make_opts(slab_group=group))
        for call in range(n):
            say("autotune slab_group=%d call %d" % (group, call))
            got = rm.fragment(*d, opts=rm.make_opts(slab_group=group, autotune=True))
            for name, a, b in zip(ref._fields, got, ref):
                assert torch.equal(a, b), (group, call, name)
    rep = [e for e in rm.autotune_report() if e["role"] == "gamma_gemm" and e["M"] == 400]
    rm.autotune_reset()
    for e in rep:
        say("Gamma M=400: %s" % e)
    # slab_group = 8: groups of 8, 8 and 4; slab_group = 4: five of 4
    assert {e["tiles"][0]: e["uses"] for e in rep} == {(128, 128): calls[8], (64, 64): 5 * calls[4]}
    for e in rep:
        assert e["best"] >= 0 and sorted(e["tiles"]) == [(64, 64), (128, 128)] and e["timed"] == [2, 2]


def test_batches_of_two_loaders():
    shapes = [(6, 40, 64), (4, 24, 50)]
    ins = [_inputs(*s) for s in shapes]
    outs = []
    rm.autotune_reset()
    for loader in (0, 1):
        frags = [dict(B=B, eps_occ=eo, eps_vir=ev, E=torch.zeros(2, dtype=torch.float64, device=B.device),
                      Gamma=torch.empty_like(B), P_ij=B.new_empty(B.shape[0], B.shape[0]),
                      P_ab=B.new_empty(B.shape[1], B.shape[1])) for B, eo, ev in ins]
        b = rm.Batch(frags, opts=rm.make_opts(autotune=True, gemm_loader=loader))
        ws = torch.empty(b.workspace_bytes, dtype=torch.uint8, device="cuda:0")
        for call in range(6):
            say("batch loader %d call %d" % (loader, call))
            b.run(ws)
            torch.cuda.synchronize()
        b.close()
        outs.append(frags)
    rep = [e for e in rm.autotune_report() if e["vec"] == 2]
    rm.autotune_reset()
    assert sorted(e["role"] for e in rep) == sorted(2 * ["ints_gemm", "gamma_gemm", "pab_gemm", "pij_gemm"])
    assert all(e["uses"] == 6 and e["timed"] == [2, 2] for e in rep)
    for f0, f1 in zip(*outs):
        for key in ("E", "Gamma", "P_ij", "P_ab"):
            assert torch.equal(f0[key], f1[key]), key
