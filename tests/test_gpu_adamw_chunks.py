"""AdamW's chunk lengths and descriptor routes: a list under 2^22 elements is cut into short chunks, one of 2^28
and more into long ones (bf16 gradients, AL8 blocks of 128-1024), up to 8 tensors travel in the kernel arguments. The same tensors stepped in a short list, in a long one (with a large tensor
beside them) and in a list of more than 8 must give the same parameters, codes and metadata bit for bit (the short
route is held to the oracle in test_gpu_adamw.py)."""
import pytest

from .gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


SIZES = [1, 255, 513, 2049, 4096 + 700, 100_003]


@pytest.mark.parametrize("grad_bf16", [True, False])
@pytest.mark.parametrize("mc", ["UF8", "FP32"])
@pytest.mark.parametrize("vc,block", [("AL8", 64), ("AL8", 128), ("AL8", 256), ("AL8", 512), ("AL8", 1024),
                                      ("AL8", 2048), ("AL16", 64), ("AL16", 256), ("AL16", 512), ("AL16", 2048),
                                      ("FP32", 256)])
def test_chunk_lengths_and_descriptor_routes_agree(dev, grad_bf16, mc, vc, block):
    import torch

    import paper_2608_22322_amd as al

    ms, vs = al.Spec(getattr(al, mc), 256), al.Spec(getattr(al, vc), block, -53.0)
    cfg = al.adamw_cfg(grad_bf16=grad_bf16, m=ms, v=vs)

    def states(sizes):
        out = []
        for i, n in enumerate(sizes):
            gen = torch.Generator(device=dev)
            gen.manual_seed(n)
            p = torch.randn(max(n, 8), generator=gen, device=dev)
            g = torch.randn(max(n, 8), generator=gen, device=dev) * 1e-3
            g *= torch.rand(max(n, 8), generator=gen, device=dev) >= 0.1
            m, mm = al.alloc_state(n, ms, dev)
            v, vm = al.alloc_state(n, vs, dev)
            out.append(al.ParamState(p, g.bfloat16() if grad_bf16 else g, 1, n, m=m, m_meta=mm, v=v, v_meta=vm))
        return out

    lists = [states(SIZES), states(SIZES + [1 << 22]), states(SIZES + [300] * 5)]
    if grad_bf16 and (mc, vc) == ("UF8", "AL8"):
        lists.append(states(SIZES + [1 << 28]))
    for sts in lists:
        arr = al.tensor_array(sts)
        ws = al.workspace(al.adamw_workspace_bytes(sts, cfg, arr=arr))
        for t in (1, 2, 3):
            al.adamw_step(sts, cfg, t, ws, arr=arr)
    for i in range(len(SIZES)):
        for name in ("param", "m", "m_meta", "v", "v_meta"):
            x = [getattr(sts[i], name) for sts in lists]
            for y in x[1:]:
                assert y is None or torch.equal(x[0], y), (SIZES[i], name)
