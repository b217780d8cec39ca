"""GPU parity of the factored steps' unit layouts: edge units (ragged rows and columns, any alignment, widths
below 8), unit heights 32 to 256, row chunks with ragged rows and flattened apply chunks."""
import pytest

from paper_2608_22322_amd.workloads import Shape, Workload

from .gpu_util import log, require_gpu
from .test_gpu_factored import F1, F2, FacPair, _spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


def _kw(al, came, uf8):
    if not came:
        return dict(vspec=_spec(al, "AL8", 256, F1))
    return dict(vspec=_spec(al, "AL16", 128, F1), mspec=_spec(al, "UF8" if uf8 else "FP32", 256, 0.0),
                cspec=_spec(al, "AL8", 512, F2))


# widths around the 8 columns of a lane, the 256 of a unit and the flattened chunk of 1024; heights around
# the 32 rows of a short list's units, the 16 of a finish group and the 4 of a batch
EDGE = [Shape(f"e{r}x{c}", r, c) for r, c in ((2, 2), (33, 3), (65, 7), (31, 8), (32, 9), (17, 15), (5, 255), (4, 257),
                                              (67, 264), (35, 519), (2, 1023), (129, 256), (37, 768), (1030, 5))]


@pytest.mark.parametrize("grad_bf16", [True, False])
@pytest.mark.parametrize("came,uf8", [(False, True), (True, True), (True, False)])
def test_edge_units_match_oracle(dev, came, uf8, grad_bf16):
    import paper_2608_22322_amd as al

    w = Workload("edges", EDGE, grad_bf16=grad_bf16, zero_frac=0.05, steps=3)
    kw = _kw(al, came, uf8)
    pair = FacPair(dev, EDGE, w, came, kw.pop("vspec"), **kw)
    for t in (1, 2, 3):
        pair.step(t)
        pair.compare(t, 1e-5 * t)


# lists of 2048 units at 64, 128 and 256 rows: the first matrix is whole units, the others ragged at that height
@pytest.mark.parametrize("rows,cols", [(8192, 4096), (8192, 8192), (16384, 8192)])
@pytest.mark.parametrize("came,uf8,grad_bf16", [(False, True, True), (False, True, False), (True, True, True),
                                                (True, True, False), (True, False, True), (True, False, False)])
def test_unit_heights_fast_sums_equal_exact(dev, rows, cols, came, uf8, grad_bf16):
    """The fast sums are kept only where they provably round as the exact ones: with AL_FLAG_EXACT_SUMS every
    mean is summed again exactly (the oracle's terms), and all states and parameters must be the same bits."""
    import torch

    import paper_2608_22322_amd as al

    shapes = [Shape("w", rows, cols), Shape("tall", 515, 256), Shape("odd", 300, 1001), Shape("slim", 700, 6),
              Shape("norm", 1, 515)]
    w = Workload("heights", shapes, grad_bf16=grad_bf16, zero_frac=0.02, steps=2)
    kw = _kw(al, came, uf8)
    v = kw.pop("vspec")
    fast = FacPair(dev, shapes, w, came, v, sample=[1, 2, 3, 4], **kw)
    exact = FacPair(dev, shapes, w, came, v, exact=True, sample=[], **kw)
    for t in (1, 2):
        fast.step(t)
        exact.step(t)
        fast.compare(t, 1e-5 * t)
        for i, (a, b) in enumerate(zip(fast.states, exact.states)):
            for name in ("param", "m", "m_meta", "v", "v_meta", "vr", "vr_meta", "vc", "vc_meta", "cr", "cr_meta",
                         "cc", "cc_meta"):
                x, y = getattr(a, name), getattr(b, name)
                assert x is None or torch.equal(x, y), f"step {t} tensor {i} {name}: exact-sums path differs"
    log(f"{rows}x{cols} came={came} uf8={uf8} bf16={grad_bf16}: fast sums equal exact sums")


# lists of whole units alone: 1025 units of 256 rows stay whole with bf16 gradients and are cut to 128 rows with
# fp32 ones; 260 units are cut to 32 rows with either
@pytest.mark.parametrize("rows,cols", [(8192, 8192), (4096, 4096)])
@pytest.mark.parametrize("came,grad_bf16", [(False, True), (False, False), (True, True), (True, False)])
def test_whole_lists_fast_sums_equal_exact(dev, rows, cols, came, grad_bf16):
    import torch

    import paper_2608_22322_amd as al

    shapes = [Shape("w", rows, cols), Shape("x", 256, 256), Shape("y", 512, 256), Shape("norm", 1, 515)]
    w = Workload("whole", shapes, grad_bf16=grad_bf16, zero_frac=0.02, steps=2)
    kw = _kw(al, came, True)
    v = kw.pop("vspec")
    fast = FacPair(dev, shapes, w, came, v, sample=[1, 2, 3], **kw)
    exact = FacPair(dev, shapes, w, came, v, exact=True, sample=[], **kw)
    for t in (1, 2):
        fast.step(t)
        exact.step(t)
        fast.compare(t, 1e-5 * t)
        for i, (a, b) in enumerate(zip(fast.states, exact.states)):
            for name in ("param", "m", "m_meta", "v", "v_meta", "vr", "vr_meta", "vc", "vc_meta", "cr", "cr_meta",
                         "cc", "cc_meta"):
                x, y = getattr(a, name), getattr(b, name)
                assert x is None or torch.equal(x, y), f"step {t} tensor {i} {name}: exact-sums path differs"
