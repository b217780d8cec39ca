"""The factored steps' 1-D tensors, stepped beside the marginal sums (short ones) or by a launch of their own: the
same body, so the same bits, and both the oracle's."""
import pytest

from paper_2608_22322_amd.workloads import Shape, Workload

from .gpu_util import log, require_gpu
from .test_gpu_factored import F1, F2, FacPair, _spec

pytestmark = pytest.mark.gpu

SMALL = [Shape("n1", 1, 777), Shape("n2", 1, 4096), Shape("n3", 1, 1), Shape("n4", 1, 256)]


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


# one past the longest that goes beside (16384 with bf16 gradients, 32768 with fp32), with and without matrices
@pytest.mark.parametrize("grad_bf16", [True, False])
@pytest.mark.parametrize("came", [False, True])
def test_beside_and_alone_give_the_same_bits(dev, came, grad_bf16):
    import torch

    import paper_2608_22322_amd as al

    line = 16384 if grad_bf16 else 32768
    kw = dict(mspec=_spec(al, "UF8", 256, 0.0), cspec=_spec(al, "AL16", 128, F2)) if came else {}
    lists = [SMALL + [Shape("long", 1, line), Shape("w", 40, 300)], SMALL + [Shape("long", 1, line + 1), Shape("w", 40, 300)], SMALL]
    pairs = []
    for shapes in lists:
        w = Workload("vec1d", shapes, grad_bf16=grad_bf16, zero_frac=0.05, steps=2)
        pairs.append(FacPair(dev, shapes, w, came, _spec(al, "AL8", 256, F1), **kw))
    for t in (1, 2):
        for pair in pairs:
            pair.step(t)
            pair.compare(t, 1e-5 * t)
        for i in range(len(SMALL)):
            for name in ("param", "m", "m_meta", "v", "v_meta"):
                x = [getattr(pair.states[i], name) for pair in pairs]
                assert x[0] is None or (torch.equal(x[0], x[1]) and torch.equal(x[0], x[2])), (t, i, name)
    log(f"came={came} bf16={grad_bf16}: 1-D tensors beside the sums and alone, same bits")
