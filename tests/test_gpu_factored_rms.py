"""The clip divisor of ragged matrices is the exactly rounded RMS(u) / d.

CAME's clipped update uhat = fl32(u / clip) is a state's input, so the RMS behind clip has to be the oracle's to the
last bit: the threshold d is chosen so that one element's u / clip lies at an fp32 rounding midpoint, on either
side of it, where an RMS an ulp off moves uhat (with beta1 = 0 the momentum is uhat itself).
"""
import math

import numpy as np
import pytest

import oracle
from paper_2608_22322_amd import data
from paper_2608_22322_amd.workloads import Shape, Workload

from .gpu_util import log, require_gpu, to_np
from .test_gpu_factored import F1, F2, FacPair, _spec

pytestmark = pytest.mark.gpu

BETA2, EPS1 = 0.999, 1e-30


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


def _grad64(g):
    g = np.asarray(g)
    return (g.astype(np.uint32) << 16).view(np.float32).astype(np.float64) if g.dtype == np.uint16 else g.astype(np.float64)


def _updates(g, rows, cols):
    """(u, RMS(u)) of the first step from zero states, in the oracle's operation order."""
    g = _grad64(g).reshape(rows, cols)
    t = g * g + EPS1
    R = np.array([np.float32((1.0 - BETA2) * (math.fsum(x) / cols)) for x in t]).astype(np.float64)
    C = np.array([np.float32((1.0 - BETA2) * (math.fsum(x) / rows)) for x in t.T]).astype(np.float64)
    u = ((1.0 / np.sqrt(R / (math.fsum(R) / rows)))[:, None] * (1.0 / np.sqrt(C))[None, :]) * g
    return u, math.sqrt(math.fsum((u * u).ravel()) / u.size)


def _thresholds(x, rms):
    """Two adjacent d, near rms / 2, between which fl32(x / (rms / d)) changes."""
    f = lambda d: np.float32(x / (rms / d))
    y = f(0.5 * rms)
    mid = 0.5 * (float(y) + float(np.nextafter(y, np.float32(np.inf))))
    d = mid * rms / x
    for _ in range(16):
        d = math.nextafter(d, 0.0)
    while f(math.nextafter(d, math.inf)) == f(d):
        d = math.nextafter(d, math.inf)
    return d, math.nextafter(d, math.inf)


# few terms, so that a rounding of any partial sum reaches the RMS: edge units with whole and shifted lanes, rows
# past the edge of a batch, widths below 8; and larger ragged ones
@pytest.mark.parametrize("grad_bf16", [True, False])
@pytest.mark.parametrize("rows,cols", [(2, 8), (3, 13), (2, 24), (5, 9), (4, 3), (40, 100), (33, 256)])
def test_clip_divisor_is_exactly_rounded(dev, rows, cols, grad_bf16):
    import torch

    import paper_2608_22322_amd as al

    shapes = [Shape("x", rows, cols)]
    tried = 0
    for seed in range(24 if rows * cols < 100 else 4):
        w = Workload("rms%d" % seed, shapes, grad_bf16=grad_bf16, zero_frac=0.0, steps=seed + 1)
        g = data.host_grad(0, w, seed + 1, np.arange(shapes[0].n))
        u, rms = _updates(g, rows, cols)
        k = int(np.argsort(u.ravel())[int(0.8 * u.size)])  # an ordinary positive update
        for d in _thresholds(float(u.ravel()[k]), rms):
            pair = FacPair(dev, shapes, w, True, _spec(al, "FP32", 256, F1), mspec=_spec(al, "FP32", 256, 0.0),
                           cspec=_spec(al, "FP32", 256, F2))
            pair.cfg.beta1, pair.cfg.clip_threshold = 0.0, d
            st, h = pair.states[0], pair.host[0]
            data.fill_grad(st.grad, 0, shapes[0], w, seed + 1)
            al.came_step(pair.states, pair.cfg, 1, pair.ws, arr=pair.arr)
            oracle.came_step(h["p"], g, rows, cols, h["m"], h["vr"], h["vc"], h["v"], h["cr"], h["cc"], 1, beta1=0.0,
                             clip_d=d)
            torch.cuda.synchronize()
            m = to_np(st.m, shapes[0].n)
            assert h["m"].codes[k] == np.float32(u.ravel()[k] / (rms / d))  # the midpoint is the oracle's
            off = np.count_nonzero(m.view(np.int32) != h["m"].codes.view(np.int32))
            assert off == 0, (seed, d, off, m[k], h["m"].codes[k])
            tried += 1
    log(f"{rows}x{cols} bf16={grad_bf16}: {tried} thresholds at a midpoint, every uhat the oracle's")
