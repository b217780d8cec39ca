"""APOLLO's projection tiles: lists with few 32-channel tiles take those, longer ones 32 * 256 / rank channels.

Every output and every channel sum is formed in the same order under both, so tensors stepped in a short list and
the same tensors beside a long one have the same bits; the long one is held to the oracle.
"""
import math

import numpy as np
import pytest

from paper_2608_22322_amd import synth

from .gpu_util import log, require_gpu
from .test_gpu_apollo import FLOOR, _run

pytestmark = pytest.mark.gpu

# channels around the tiles of 32, 64 and 128, projected lengths around a slice of 16
SMALL = [(33, 16), (65, 17), (129, 31), (40, 127), (257, 256), (128, 128), (5, 130)]


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


def _step(al, dev, shapes, rank, bf16):
    """State tensors after two steps over the list."""
    import torch

    mspec, vspec = al.Spec(al.UF8, 256), al.Spec(al.AL8, 256, FLOOR)
    cfg = al.apollo_cfg(lr=1e-4, gamma=1.01, rank=rank, grad_bf16=bf16, m=mspec, v=vspec, weight_decay=0.01)
    items = []
    for i, (rows, cols) in enumerate(shapes):
        n = rank * max(rows, cols)
        p = torch.from_numpy(synth.normal_f32(synth.param_key(i), rows * cols, 0.02)).to(dev)
        g = torch.empty(rows * cols, dtype=torch.bfloat16 if bf16 else torch.float32, device=dev)
        pj = torch.empty(min(rows, cols) * rank, dtype=torch.float32, device=dev)
        al.synth_normal(pj, synth.proj_key(i, 0), 1.0 / math.sqrt(rank))
        items.append((p, g, rows, cols, pj, *al.alloc_state(n, mspec, dev), *al.alloc_state(n, vspec, dev),
                      torch.zeros(4, device=dev)))
    arr = al.apollo_tensor_array(items)
    ws = al.workspace(al.apollo_workspace_bytes(arr, len(items), cfg), dev)
    for t in (1, 2):
        for i, it in enumerate(items):
            al.synth_normal(it[1], synth.grad_key(i, t), 1e-3)
        al.apollo_step(arr, len(items), cfg, t, ws)
    torch.cuda.synchronize()
    return [[x for x in (it[0], *it[5:])] for it in items]


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("rank", [64, 128])
def test_tile_heights_give_the_same_bits(dev, rank, bf16):
    import torch

    import paper_2608_22322_amd as al

    short = _step(al, dev, SMALL, rank, bf16)
    long_ = _step(al, dev, SMALL + [(32 * (256 * 128 // rank), 16)], rank, bf16)  # past the line by the small ones
    for shape, a, b in zip(SMALL, short, long_):
        for k, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), (shape, k)
    log(f"rank {rank} bf16 {bf16}: same bits under both tile heights")


@pytest.mark.parametrize("rank", [64, 128])
def test_long_lists_match_the_oracle(dev, rank):
    n = 32 * (256 * 128 // rank)
    _run(dev, [(n + 1, 18), (33, 16), (130, 70), (70, 129)], rank, rank == 64, coded=True, steps=2)
