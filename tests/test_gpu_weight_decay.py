"""GPU parity of the factored steps' parameter update with a weight decay, on every layout of the apply passes.

The updates are binary64, rounded once to fp32 (CAME's whole 256 x 256 units apart), from factors formed by the
oracle's own operations, so the parameters are the oracle's bits: a value could differ only where its binary64
forms straddle an fp32 rounding midpoint, at a few 2^-53 of relative difference about one value in 2^26. CAME's
whole units form the change of p in fp32 (at most 2^-22 of it) and round p once.
"""
import numpy as np
import pytest

import oracle
from paper_2608_22322_amd import data
from paper_2608_22322_amd.workloads import Shape, Workload

from .gpu_util import compare_bits, log, require_gpu, to_np
from .test_gpu_factored import F1, F2, FacPair, _spec

pytestmark = pytest.mark.gpu

LR, WD = 1e-4, 0.01

# ragged rows at a width that is a multiple of 256, ragged columns of any alignment, widths below the 4 of a
# lane and the 8 of an edge unit, a chunk boundary inside a row, 1-D
RAGGED = [Shape("rows", 300, 512), Shape("odd", 130, 513), Shape("even", 300, 66), Shape("slim", 257, 3),
          Shape("flat", 2, 1030), Shape("tall", 700, 256), Shape("norm", 1, 777)]
WHOLE = [Shape("w", 256, 512), Shape("x", 512, 768)]


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


def _pair(al, dev, shapes, w, came, uf8):
    if came:
        pair = FacPair(dev, shapes, w, True, _spec(al, "FP32", 256, F1), mspec=_spec(al, "UF8" if uf8 else "FP32", 256, 0.0),
                       cspec=_spec(al, "FP32", 256, F2))
    else:
        pair = FacPair(dev, shapes, w, False, _spec(al, "FP32", 256, F1))
    pair.cfg.lr, pair.cfg.weight_decay = LR, WD
    return pair


def _step(al, pair, t):
    """A step of the pair on the GPU and, with the same learning rate and decay, on the host."""
    import torch

    for i, (s, st) in enumerate(zip(pair.shapes, pair.states)):
        data.fill_grad(st.grad, i, s, pair.w, t)
        h, g = pair.host[i], data.host_grad(i, pair.w, t, np.arange(s.n))
        if pair.came:
            oracle.came_step(h["p"], g, s.rows, s.cols, h["m"], h["vr"], h["vc"], h["v"], h["cr"], h["cc"], t, lr=LR,
                             wd=WD)
        else:
            oracle.adafactor_step(h["p"], g, s.rows, s.cols, h["vr"], h["vc"], h["v"], t, lr=LR, wd=WD)
    (al.came_step if pair.came else al.adafactor_step)(pair.states, pair.cfg, t, pair.ws, arr=pair.arr)
    torch.cuda.synchronize()


@pytest.mark.parametrize("grad_bf16", [True, False])
@pytest.mark.parametrize("came,uf8", [(False, False), (True, False), (True, True)])
def test_ragged_parameters_are_the_binary64_update(dev, came, uf8, grad_bf16):
    import paper_2608_22322_amd as al

    w = Workload("decay", RAGGED, grad_bf16=grad_bf16, zero_frac=0.05, steps=3)
    pair = _pair(al, dev, RAGGED, w, came, uf8)
    n = sum(s.n for s in RAGGED)
    for t in (1, 2, 3):
        _step(al, pair, t)
        assert pair.compare(t, 1e-5 * t) == 0  # no code differs either, so neither does a momentum
        diff = 0
        for i, s in enumerate(RAGGED):
            g, o = to_np(pair.states[i].param, s.n).view(np.int32), pair.host[i]["p"].view(np.int32)
            assert np.abs(g.astype(np.int64) - o).max() <= 1, (t, s.name)
            diff += int(np.count_nonzero(g != o))
        assert diff <= 1 + n * 2.0 ** -20, (t, diff)
        log(f"came={came} uf8={uf8} bf16={grad_bf16} t{t}: {diff} of {n} parameters an ulp off")


@pytest.mark.parametrize("grad_bf16", [True, False])
def test_came_whole_unit_parameters(dev, grad_bf16):
    """Per step at most an ulp of p (its rounding, on both sides half of one) and 2^-22 of the two parts of the
    change, |update| <= |change| + lr wd |p| and lr wd |p|; the errors of the steps add."""
    import paper_2608_22322_amd as al

    w = Workload("decay", WHOLE, grad_bf16=grad_bf16, zero_frac=0.05, steps=3)
    pair = _pair(al, dev, WHOLE, w, True, False)
    lim = [np.zeros(s.n) for s in WHOLE]
    for t in (1, 2, 3):
        before = [h["p"].copy() for h in pair.host.values()]
        _step(al, pair, t)
        assert pair.compare(t, 1e-5 * t) == 0
        for i, s in enumerate(WHOLE):
            g, o = to_np(pair.states[i].param, s.n).astype(np.float64), pair.host[i]["p"]
            big = np.maximum(np.abs(o), np.abs(before[i]))
            lim[i] += np.spacing(big) + 2.0 ** -22 * (np.abs(o.astype(np.float64) - before[i]) + 2 * LR * WD * big)
            assert np.all(np.abs(g - o) <= lim[i]), (t, s.name)


@pytest.mark.parametrize("shapes", [RAGGED, WHOLE], ids=["ragged", "whole"])
def test_came_decay_without_gradients(dev, shapes):
    """lr wd = 1e-6, no gradients: every step is p <- fl32(p (1 - lr wd)), bit for bit; in whole units up to the
    values whose change, rounded to fp32, moves them over a midpoint: 2^-22 of 1e-6 |p| against half an ulp of at
    least 2^-25 |p|, at most 8e-6 of the values per step, an ulp each."""
    import torch

    import paper_2608_22322_amd as al

    w = Workload("decay", shapes, grad_bf16=False, zero_frac=0.0, steps=40)
    pair = _pair(al, dev, shapes, w, True, True)
    p = [to_np(st.param, s.n).copy() for s, st in zip(shapes, pair.states)]
    for st in pair.states:
        st.grad.zero_()
    for t in range(1, 41):
        al.came_step(pair.states, pair.cfg, t, pair.ws, arr=pair.arr)
        p = [(x.astype(np.float64) * (1.0 - LR * WD)).astype(np.float32) for x in p]
    torch.cuda.synchronize()
    for s, st, x in zip(shapes, pair.states, p):
        g = to_np(st.param, s.n)
        if shapes is RAGGED:
            compare_bits(g, x, s.name)
        else:
            off = np.abs(g.view(np.int32).astype(np.int64) - x.view(np.int32))
            log(f"{s.name}: {np.count_nonzero(off)} of {s.n} values off after 40 steps, at most {off.max()} ulp")
            assert np.count_nonzero(off) <= 40 * 8e-6 * s.n and off.max() <= 2
