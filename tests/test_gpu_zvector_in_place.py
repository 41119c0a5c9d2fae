"""rimp2_zvector's result may lie over one of its inputs (a caller that needs L'
or L'' no longer): D_ai is first written after the last read of L1 and L2.  Bit
for bit against a result array of its own, over several workgroups of the
right-hand side's kernel, which write while others still read."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2410_21888_amd as rm
from paper_2410_21888_amd import gradient as G
from gpu_util import to_dev, say
from test_gpu_response import full_factor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["L1", "L2"])
def test_result_over_an_input(over):
    nocc, nvir, naux = 9, 60, 50
    nmo = nocc + nvir
    Bf, eo, ev = full_factor(nocc, nvir, naux, 21)
    rng = np.random.default_rng(22)
    a = dict(zip(("Bf", "eo", "ev", "Pij", "Pab", "L1", "L2"),
                 to_dev(Bf, eo, ev, np.eye(nocc), np.eye(nvir), rng.standard_normal((nocc, nmo)),
                        rng.standard_normal((nvir, nmo)))))
    say("zvector result over %s" % over)
    ref, it, _ = G.zvector(*a.values())
    L = G._L()
    n = ctypes.c_size_t(0)
    assert L.rimp2_zvector_workspace_size(nocc, nvir, naux, ctypes.byref(n)) == rm.RIMP2_OK
    ws = torch.empty(n.value, dtype=torch.uint8, device="cuda:0")
    its = ctypes.c_int32(0)
    rc = L.rimp2_zvector(nocc, nvir, naux, *(t.data_ptr() for t in a.values()), a[over].data_ptr(), 1e-12, 500,
                         ctypes.byref(its), None, ws.data_ptr(), n.value, torch.cuda.current_stream().cuda_stream)
    assert rc == rm.RIMP2_OK and its.value == it
    assert torch.equal(a[over].reshape(-1)[: nocc * nvir], ref.reshape(-1))
