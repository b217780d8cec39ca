"""APOLLO's update is the same binary64 expression, p (1 - lr wd) - lr g (s_c / lam), on whole and ragged tensors.

A tensor of whole 256 x 256 units and the same tensor with one more channel, of zero gradients, have the same channel
scales and the same limiter, bit for bit. The first step from p = 0 gives p1 = -fl32(lr g (s_c / lam)); a step from
p = -p1 then leaves what the fp32 rounding of that product dropped: its binary64 bits beyond the 24th, so the two
layouts' results agree only if the products do to their last bits.
"""
import numpy as np
import pytest

from paper_2608_22322_amd import synth

from .gpu_util import log, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


def _step(al, dev, p, g, proj, rank, bf16):
    """One step (t = 2, the limiter active) from zero moments; p in place."""
    import torch

    rows, cols = g.shape
    n = rank * max(rows, cols)
    spec = al.Spec(al.FP32, 256)
    m, v = al.alloc_state(n, spec, dev)[0], al.alloc_state(n, spec, dev)[0]
    ns = torch.full((4,), 1e-3, dtype=torch.float32, device=dev)
    gd = g.to(torch.bfloat16 if bf16 else torch.float32).contiguous().view(-1)
    cfg = al.apollo_cfg(lr=1e-2, gamma=1.01, rank=rank, grad_bf16=bf16, m=spec, v=spec)
    arr = al.apollo_tensor_array([(p, gd, rows, cols, proj, m, None, v, None, ns)])
    al.apollo_step(arr, 1, cfg, 2, al.workspace(al.apollo_workspace_bytes(arr, 1, cfg), dev))
    torch.cuda.synchronize()
    assert abs(float(ns[0]) / (1.01 * (1e-3 + 1e-8)) - 1) < 1e-6  # the limiter divided: n / lam = gamma (prev + 1e-8)


@pytest.mark.parametrize("rank", [64, 256])
@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("rows,cols", [(512, 256), (256, 768)])
def test_ragged_update_is_the_whole_units_one(dev, rows, cols, bf16, rank):
    import torch

    import paper_2608_22322_amd as al

    g = torch.from_numpy(synth.normal_f32(synth.grad_key(0, 1), rows * cols, 1e-3).reshape(rows, cols)).to(dev)
    right = rows >= cols
    wide = torch.zeros((rows + 1, cols) if right else (rows, cols + 1), device=dev)
    wide[:rows, :cols] = g
    proj = torch.empty(min(rows, cols) * rank, dtype=torch.float32, device=dev)
    al.synth_normal(proj, synth.proj_key(0, 0), 1.0 / np.sqrt(rank))
    out = []
    for x in (g, wide):
        p = torch.zeros(x.numel(), device=dev)
        _step(al, dev, p, x, proj, rank, bf16)
        q = -p
        _step(al, dev, q, x, proj, rank, bf16)
        out.append((p.view(x.shape)[:rows, :cols].contiguous(), q.view(x.shape)[:rows, :cols].contiguous()))
    for a, b, what in zip(out[0], out[1], ("product", "its dropped bits")):
        off = int((a.view(torch.int32) != b.view(torch.int32)).sum())
        assert off == 0, f"{what}: {off} of {a.numel()} differ"
    left = int((out[0][1] != 0).sum())
    assert left > 0.9 * rows * cols  # the second step does leave the dropped bits
    log(f"{rows}x{cols} r{rank} bf16={bf16}: {left} remainders, all the same")
