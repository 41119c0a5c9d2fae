"""The Z-vector's CG on vectors longer than what its step kernel holds in
registers (8192 elements) and on odd lengths, by the residual that the
antisymmetrised term gives for the solution (here by matrix products, which are
held against the oracle's sums at a small size).

Bound: the residual CG stops at (1e-13) plus the rounding of one application,
sums of up to nov naux = 1.7e5 terms in float64 (about sqrt(1.7e5) 1.1e-16 of
the operator's result) times its condition number (orbital gaps from 0.4 to 25,
about 60): 3e-12 at most, 1e-11 asked.
"""
import numpy as np
import pytest
import torch

from oracle import rimp2_oracle as O
import paper_2410_21888_amd as rm
from paper_2410_21888_amd import gradient as G
from gpu_util import to_dev, say
from test_gpu_response import full_factor

pytestmark = pytest.mark.gpu


def antisym(Bf, D):
    c = np.tensordot(Bf, D, ((0, 1), (0, 1)))
    Y = np.tensordot(D, Bf, ((0,), (0,)))                      # [s][q][P]
    return 2.0 * Bf @ c - np.tensordot(Bf, Y, ((1, 2), (0, 2)))


@pytest.mark.parametrize("shape", [(64, 128, 12), (57, 145, 20), (9, 3, 40), (11, 93, 33)])
def test_zvector_residual(shape):
    nocc, nvir, naux = shape
    nmo = nocc + nvir
    Bf, eo, ev = full_factor(nocc, nvir, naux, sum(shape), scale=0.01)
    rng = np.random.default_rng(sum(shape) + 5)
    L1, L2 = rng.standard_normal((nocc, nmo)), rng.standard_normal((nvir, nmo))
    s, D = Bf[:7, :7], rng.standard_normal((7, 7))
    np.testing.assert_allclose(antisym(s, D), O.antisym_term(s, D), rtol=1e-12, atol=1e-12 * np.abs(s).max() ** 2)
    say("zvector residual %s" % (shape,))
    D_ai, it, res = G.zvector(*to_dev(Bf, eo, ev, np.eye(nocc), np.eye(nvir), L1, L2), tol=1e-13, max_iter=400)
    assert res <= 1e-13
    x = D_ai.cpu().numpy()
    Dv = np.zeros((nmo, nmo))
    Dv[nocc:, :nocc] = x
    rhs = L2[:, :nocc] - L1[:, nocc:].T - antisym(Bf, np.eye(nmo))[nocc:, :nocc]
    r = rhs - (ev[:, None] - eo[None, :]) / 2.0 * x - antisym(Bf, Dv)[nocc:, :nocc]
    rel = np.linalg.norm(r) / np.linalg.norm(rhs)
    say("  %d iterations, residual of the solution %.2e" % (it, rel))
    assert rel <= 1e-11


@pytest.mark.parametrize("tol", [1e-2, 1e-4, 1e-6, 1e-8, 1e-10])
def test_zvector_stops_where_it_converges(tol):
    """Iterations are queued four at a time: whatever remainder the last one falls on,
    a limit of just as many gives the same bits, and one fewer is too few."""
    nocc, nvir, naux = 6, 30, 64
    nmo = nocc + nvir
    Bf, eo, ev = full_factor(nocc, nvir, naux, 7)
    rng = np.random.default_rng(8)
    args = to_dev(Bf, eo, ev, np.eye(nocc), np.eye(nvir), rng.standard_normal((nocc, nmo)),
                  rng.standard_normal((nvir, nmo)))
    D, it, res = G.zvector(*args, tol=tol)
    say("zvector tol %g: %d iterations" % (tol, it))
    assert it >= 1 and res <= tol
    D2, it2, res2 = G.zvector(*args, tol=tol, max_iter=it)
    assert it2 == it and res2 == res and torch.equal(D, D2)
    if it > 1:
        with pytest.raises(rm.Rimp2Error) as ei:
            G.zvector(*args, tol=tol, max_iter=it - 1)
        assert ei.value.code == rm.RIMP2_ENOCONV
