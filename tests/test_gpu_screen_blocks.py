"""The screening kernels at the edges of their blocks, against the oracle:
samples in blocks of 16 over at most 256 (gradient) or 1024 (forward)
workgroups, so that a workgroup takes none, one or several blocks and the
last one is ragged; pair features over 16 x 16 pairs and 64 columns; and the
budgeted threshold against the bisection it stands for.  FP64 sums in another
order: 1e-12 relative (norms)."""
import numpy as np
import pytest
import torch

import synth
from oracle import screen_oracle as S
from paper_2410_21888_amd import screen as SC
from gpu_util import to_dev, rel_fro, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, 4096, 4113, 16384 + 5])
def test_network_blocks(n):
    rng = np.random.default_rng(n)
    x, t, p = rng.standard_normal((n, 4)), rng.standard_normal(n), rng.standard_normal(S.NP) * 0.3
    say("network n=%d" % n)
    dx, dt, dp = to_dev(x, t, p)
    assert rel_fro(SC.mlp_forward(dx, dp).cpu().numpy(), S.forward(x, p)) <= 1e-12
    loss, grad = SC.mlp_loss_grad(dx, dt, dp)
    L, g = S.loss_grad(x, t, p)
    assert abs(float(loss) - L) <= 1e-12 * L
    assert rel_fro(grad.cpu().numpy(), g) <= 1e-12


@pytest.mark.parametrize("shape", [(1, 1, 1), (15, 3, 31), (16, 5, 64), (17, 6, 65), (33, 9, 130)])
def test_feature_blocks(shape):
    f = synth.screen_system(4000 + shape[0], nocc=shape[0], nvir=shape[1], naux=shape[2])
    B, eo, ev = f.arrays()
    r, _ = f.positions()
    say("features %s" % (shape,))
    feat, bd = SC.pair_features(*to_dev(B, eo, ev, r))
    assert rel_fro(feat.cpu().numpy(), S.pair_features(B, eo, r)) <= 1e-12
    assert rel_fro(bd.cpu().numpy(), S.pair_bound(B, eo, ev)) <= 1e-12


@pytest.mark.parametrize("nocc,budget", [(1, 1e-6), (5, 1e-6), (33, 1e-7), (33, 10.0), (40, 0.0)])
def test_budget_threshold_is_the_bisection(nocc, budget):
    pred = torch.from_numpy(np.random.default_rng(nocc).uniform(-12, -4, nocc * nocc)).to("cuda:0")
    lo, hi = -30.0, 0.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        if float(SC.screen_mask(pred, nocc, mid)[1]) <= budget:
            lo = mid
        else:
            hi = mid
    assert SC.budget_threshold(pred, nocc, budget) == lo


@pytest.mark.parametrize("n,batch,steps", [(50, 17, 1), (300, 64, 8), (300, 300, 9), (700, 5000, 17)])
def test_fit_is_its_single_steps(n, batch, steps):
    """Trainer.fit (steps in a row, rows gathered in the kernel) against the
    same steps through mlp_loss_grad and adam on written-out minibatches: the
    same sums in the same order, bit for bit; step counts around an upload."""
    rng = np.random.default_rng(n + steps)
    dx, dt, p = to_dev(rng.standard_normal((n, 4)), rng.standard_normal(n), rng.standard_normal(S.NP) * 0.3)
    say("fit n=%d batch=%d steps=%d" % (n, batch, steps))
    q, m, v = p.clone(), torch.zeros_like(p), torch.zeros_like(p)
    tr = SC.Trainer(p.clone(), lr=1e-2)
    last = tr.fit(dx, dt, steps=steps, batch=batch, seed=3)
    draw, loss = np.random.default_rng(3), None
    for k in range(steps):
        idx = torch.from_numpy(draw.choice(n, size=min(batch, n), replace=False)).to("cuda:0")
        loss, grad = SC.mlp_loss_grad(dx.index_select(0, idx), dt.index_select(0, idx), q)
        SC.adam(grad, q, m, v, k + 1, 1e-2)
    assert tr.step == steps and float(loss) == last
    assert torch.equal(tr.params, q) and torch.equal(tr.m, m) and torch.equal(tr.v, v)
