"""The codecs' two chunk lengths: arrays of 2^21 and more elements (AL16: 2^22 encoding, 7 * 2^20 decoding) take
2048-element chunks, shorter ones max(block, 256). The same values must give the same codes, metadata and decoded values through both (the short
path is held to the oracle in test_gpu_codec.py), ragged ends included."""
import pytest

from .gpu_util import require_gpu

pytestmark = pytest.mark.gpu

LONG = 2048 * 1024


@pytest.fixture(scope="module")
def dev():
    require_gpu()
    import torch

    return torch.device("cuda:0")


@pytest.mark.parametrize("codec", ["AL8", "AL16", "UF8"])
@pytest.mark.parametrize("block", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("tail", [0, 1, 2047, 700])
def test_long_and_short_chunks_agree(dev, codec, block, tail):
    _long_and_short(dev, codec, block, LONG + tail, tail)


@pytest.mark.parametrize("block", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("tail", [0, 1, 700])
def test_al16_long_and_short_chunks_agree(dev, block, tail):
    _long_and_short(dev, "AL16", block, (7 << 20) + tail, tail)


def _long_and_short(dev, codec, block, n, tail):
    import torch

    import paper_2608_22322_amd as al

    c = getattr(al, codec)
    gen = torch.Generator(device=dev)
    gen.manual_seed(block + tail)
    x = torch.randn(n, generator=gen, device=dev)
    if codec != "UF8":
        x = torch.exp2(-20 + 4 * x)
        x[: 5 * block] = 0.0  # blocks without a positive value
        x[7 * block: 8 * block] = 3e-6  # one value
    x *= torch.rand(n, generator=gen, device=dev) >= 0.05
    spec = al.Spec(c, block, -53.0)

    def both(y):
        codes, meta = al.alloc_state(y.numel(), spec, dev)
        codes.fill_(7)
        al.quantize(c, y, block, -53.0, codes, meta)
        out = torch.full((y.numel() + 4,), -1.0, device=dev)
        al.dequantize(c, codes, meta, y.numel(), block, out)
        assert torch.all(out[y.numel():] == -1.0)
        return codes, meta, out[: y.numel()]

    codes, meta, out = both(x)
    half = (n // 2) // 2048 * 2048
    per = 1 if codec == "UF8" else 2
    for lo, hi in ((0, half), (half, n)):
        sc, sm, so = both(x[lo:hi].clone())
        nb = (hi - lo + block - 1) // block
        assert torch.equal(sc, codes[lo: lo + nb * block])
        assert torch.equal(sm[: per * nb], meta[per * (lo // block): per * (lo // block + nb)])
        assert torch.equal(so, out[lo:hi])


@pytest.mark.parametrize("block", [64, 2048])
def test_uf8_arrays_past_the_cache_agree_with_shorter_ones(dev, block):
    """2^26 values and more are read past the last-level cache: the same codes as their parts, a ragged end included."""
    import torch

    import paper_2608_22322_amd as al

    n = (1 << 26) + 700
    x = torch.randn(n, generator=torch.Generator(device=dev).manual_seed(block), device=dev)
    spec = al.Spec(al.UF8, block)
    codes, meta = al.alloc_state(n, spec, dev)
    al.quantize(al.UF8, x, block, 0.0, codes, meta)
    for lo, hi in ((0, 1 << 22), (n // 2048 * 2048 - (1 << 21), n)):
        part = x[lo:hi].clone()
        sc, sm = al.alloc_state(hi - lo, spec, dev)
        al.quantize(al.UF8, part, block, 0.0, sc, sm)
        nb = (hi - lo + block - 1) // block
        assert torch.equal(sc[: nb * block], codes[lo: lo + nb * block])
        assert torch.equal(sm[:nb], meta[lo // block: lo // block + nb])
