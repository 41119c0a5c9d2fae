"""Trainer.fit refuses, on the host and before anything is launched, inputs that
its kernels would read out of range: a target vector shorter than the rows, one
on another device, narrower types, rows of another width, short parameters."""
import pytest
import torch

from paper_2410_21888_amd import screen as SC

N = 40


def _good():
    f64 = dict(dtype=torch.float64)
    return dict(x=torch.zeros(N, 4, **f64), t=torch.zeros(N, **f64), params=torch.zeros(SC.N_PARAMS, **f64))


BAD = {
    "short t": (dict(t=torch.zeros(N - 1, dtype=torch.float64)), "one target"),
    "two targets a row": (dict(t=torch.zeros(N, 2, dtype=torch.float64)), "one target"),
    "scalar t": (dict(t=torch.zeros((), dtype=torch.float64)), "one target"),
    "t on another device": (dict(t=torch.zeros(N, dtype=torch.float64, device="meta")), "t is on meta"),
    "float32 t": (dict(t=torch.zeros(N)), "t must be float64"),
    "float32 x": (dict(x=torch.zeros(N, 4)), "x must be float64"),
    "three features": (dict(x=torch.zeros(N, 3, dtype=torch.float64)), "four features"),
    "params on another device": (dict(params=torch.zeros(SC.N_PARAMS, dtype=torch.float64, device="meta")),
                                 "params is on meta"),
    "short params": (dict(params=torch.zeros(SC.N_PARAMS - 1, dtype=torch.float64)), "parameters"),
    "host tensors": ({}, "on the GPU"),
}


@pytest.mark.parametrize("case", sorted(BAD))
def test_fit_refuses(case):
    change, message = BAD[case]
    a = {**_good(), **change}
    tr = SC.Trainer(a["params"])
    with pytest.raises(ValueError, match=message):
        tr.fit(a["x"], a["t"], steps=3, batch=8)
    assert tr.step == 0


@pytest.mark.gpu
def test_fit_takes_a_target_column_and_spare_targets():
    """Shapes that hold one target a row without being [n], and targets past the
    last row, train as the plain vector does."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    kw = dict(dtype=torch.float64, device="cuda:0", generator=gen)
    x, t = torch.randn(N, 4, **kw), torch.randn(N + 3, **kw)
    runs = []
    for target in (t[:N].clone(), t[:N].reshape(N, 1), t):
        tr = SC.Trainer(SC.init_params(2, "cuda:0"))
        tr.fit(x, target, steps=3, batch=16, seed=1)
        runs.append(tr.params)
    assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2])
