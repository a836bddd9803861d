"""bf16 decode against the fp32 decode of the same planes, bit for bit: the fp32
value rounded to nearest even, in every order of the tiles (runs of
neighbouring tiles, strided), and for values that are not finite."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import paper_2607_08643_amd as bsq
from parity_bounds import say

pytestmark = pytest.mark.gpu


def random_layer(cfg, n_mats, d_out, d_in, gpu):
    g = torch.Generator(device=gpu).manual_seed(5)
    L = bsq.layer_empty(cfg, d_out, d_in, n_mats, gpu)
    for s in range(cfg.stages):
        L.codes[s].random_(*((0, 256) if cfg.b == 8 else (-32768, 32768)), generator=g)
        L.gains[s].uniform_(-1.0, 1.0, generator=g)
    return L


def codec(cfg, gpu, b2=None):
    g = torch.Generator(device=gpu).manual_seed(9)
    rnd = lambda *s: torch.randn(s, generator=g, device=gpu)  # noqa: E731
    decs = [SimpleNamespace(W1=rnd(cfg.hidden, cfg.b), b1=rnd(cfg.hidden), W2=rnd(cfg.d, cfg.hidden),
                            b2=rnd(cfg.d) if b2 is None else b2,
                            E=rnd(cfg.b, cfg.d) if cfg.encoder else None) for _ in range(cfg.stages)]
    return bsq.bsq_codec_prepare(cfg, decs, gpu)


def rounded(f32):
    """fp32 bits to bf16 bits: nearest even, infinities kept, NaN quiet with
    its upper payload bits kept."""
    u = f32.view(torch.int32).long() & 0xFFFFFFFF
    near = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) & 0xFFFF
    special = (u >> 16) | torch.where((u & 0xFFFF) != 0, 0x40, 0)
    return torch.where((u & 0x7F800000) == 0x7F800000, special, near)


# more blocks than tiles; runs of two lengths (1024 // n_mats blocks a matrix);
# a stack larger than the block count; runs of 16 tiles, which are halved
SHAPES = [(1, 200, 520), (6, 704, 2056), (1500, 64, 136), (128, 512, 2048)]


@pytest.mark.parametrize("n_mats,d_out,d_in", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("b,stages", [(8, 1), (8, 3), (16, 1), (16, 2)])
def test_bf16_decode_equals_rounded_fp32_decode(b, stages, n_mats, d_out, d_in, gpu):
    say(f"decode order b={b} stages={stages} {n_mats}x{d_out}x{d_in}")
    cfg = bsq.Config(d=8, stages=stages, hidden=8, protect_num=0, codebook_bits=b,
                     encoder=bsq.ENC_LINEAR if b == 16 else bsq.ENC_IDENTITY)
    cd, L = codec(cfg, gpu), random_layer(cfg, n_mats, d_out, d_in, gpu)
    f = bsq.bsq_decode(cfg, cd, L, dtype=torch.float32)
    h = torch.full_like(f, -1.0, dtype=torch.bfloat16)
    bsq.bsq_decode(cfg, cd, L, out=h)
    assert torch.equal(h.view(torch.int16), f.to(torch.bfloat16).view(torch.int16))


@pytest.mark.parametrize("b", [8, 16])
def test_bf16_decode_of_values_that_are_not_finite(b, gpu):
    """Decoder tables with infinities and NaNs of several payloads (a diverged
    codec): the bf16 bits are those of the fp32 decode, rounded."""
    say(f"decode non-finite b={b}")
    cfg = bsq.Config(d=8, stages=1, hidden=8, protect_num=0, codebook_bits=b,
                     encoder=bsq.ENC_LINEAR if b == 16 else bsq.ENC_IDENTITY)
    bits = np.array([0x7F800000, 0xFF800000, 0x7FC00000, 0x7FC00001, 0xFFC12345, 0x7FFFFFFF, 0x7F7FFFFF, 0x3F800000],
                    dtype=np.uint32)
    cd, L = codec(cfg, gpu, torch.from_numpy(bits.view(np.float32)).to(gpu)), random_layer(cfg, 1, 100, 264, gpu)
    f = bsq.bsq_decode(cfg, cd, L, dtype=torch.float32)
    h = bsq.bsq_decode(cfg, cd, L, dtype=torch.bfloat16)
    assert not torch.isfinite(f).all()
    assert torch.equal(h.view(torch.int16).long() & 0xFFFF, rounded(f))
