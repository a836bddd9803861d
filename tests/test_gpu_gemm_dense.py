"""The decode-once GEMM (many tokens) against the oracle, at the edges of its
tiles, for every (d, stages), payload format and output layout, with the
per-output bars of parity_bounds."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_08643_amd as bsq
import synth
from parity_bounds import check_close, product_floor, say
from test_gpu_parity import decoders, ocfg

pytestmark = pytest.mark.gpu

# (M, d_out, d_in, config, rank): blocks of 128 x 128 (few blocks), 256 x 128,
# 256 x 192 and 256 x 256 (tokens x rows) with ragged last tiles
CASES = [
    (2049, 130, 1000, dict(d=8, hidden=8, stages=3, protect_format=bsq.PROT_E4M3), 16),
    (1100, 200, 1072, dict(d=16, hidden=16, protect_format=bsq.PROT_E5M2), 0),
    (1537, 64, 528, dict(d=16, hidden=16, stages=4, protect_num=1, protect_den=9), 5),
    (1024, 61, 264, dict(d=8, hidden=8, stages=4, protect_num=0), 0),
    (2040, 4090, 136, dict(d=8, hidden=8), 16),
    (2000, 12250, 72, dict(d=8, hidden=8, stages=1), 3),
    (2048, 8192, 80, dict(d=16, hidden=16, stages=1), 16),
    (2048, 5000, 48, dict(d=16, hidden=16, stages=3), 1),
    # few tokens of many rows at d = 8, and of any at d = 16
    (129, 4100, 264, dict(d=8, hidden=8), 16),
    (65, 100, 400, dict(d=16, hidden=16), 16),
    # K split over blocks
    (1030, 260, 3000, dict(d=8, hidden=8), 16),
    (1025, 513, 2608, dict(d=16, hidden=16), 0),
]


@pytest.mark.parametrize("M,d_out,d_in,kw,rank", CASES, ids=[f"{c[0]}x{c[1]}x{c[2]}-d{c[3]['d']}" for c in CASES])
def test_many_tokens_match_oracle(M, d_out, d_in, kw, rank, gpu):
    say(f"dense gemm M={M} {d_out}x{d_in} {kw} rank={rank}")
    cfg = bsq.Config(**kw)
    oc = ocfg(cfg)
    decs = decoders(cfg, seed=5)
    W, _ = synth.weight(d_out, d_in, seed=7, k_outliers=cfg.k(d_in), device=gpu)
    codec = bsq.bsq_codec_prepare(cfg, decs, device=gpu)
    layer = bsq.bsq_encode(cfg, codec, W)
    X = synth.activation(d_in, seed=8, device=gpu, batch=M)
    lora = lref = None
    if rank:
        A, B = synth.lora(d_out, d_in, rank, seed=9, device=gpu)
        lref = (oracle.to_f32(A), oracle.to_f32(B))
        flat = torch.empty(A.numel() + 1, dtype=A.dtype, device=gpu)  # A at an odd element: two-byte loads
        odd = flat[1:].view(A.shape).copy_(A) if rank == 5 else A
        lora = (odd, B)
    Y = bsq.bsq_gemm(cfg, codec, layer, X, lora=lora, y_dtype=torch.float32)
    # bf16 rows of an odd pitch, and activations of a longer pitch, in one more call
    wide = torch.empty((M, d_out + 3), dtype=torch.bfloat16, device=gpu)[:, :d_out]
    Xw = torch.empty((M, d_in + 8), dtype=torch.bfloat16, device=gpu)[:, :d_in].copy_(X)
    Yb = bsq.bsq_gemm(cfg, codec, layer, Xw, lora=lora, out=wide)
    torch.cuda.synchronize()
    tabs = oracle.decoder_table(oc, decs)
    enc = oracle.encode(oc, decs, oracle.to_f32(W), tables=tabs)
    w_hat = oracle.decode(oc, decs, enc, tables=tabs)
    Xf = oracle.to_f32(X)
    ref = oracle.dense_product(w_hat, Xf, lref)
    floor = product_floor("gemm", cfg.d, enc, tabs, w_hat, Xf, lref)
    check_close(Y.cpu().numpy(), ref, 2e-2, "fp32 out", floor)
    check_close(Yb.float().cpu().numpy(), ref, 2e-2, "bf16 out, odd pitches", floor, out_bf16=True)
    assert torch.equal(Yb, Y.to(torch.bfloat16)), "the two layouts give different sums"


def test_row_slabs_agree_with_their_rows_alone(gpu):
    """A layer decoded in several slabs: its rows equal the product of those
    rows as a layer of their own, up to the order of 5,200 fp32 additions (a
    misplaced row would differ by about the rms)."""
    M, d_out, d_in = 1024, 57408, 5120
    say(f"dense gemm slabs M={M} {d_out}x{d_in}")
    cfg = bsq.Config(d=8, hidden=8)
    codec = bsq.bsq_codec_prepare(cfg, decoders(cfg, seed=3), device=gpu)
    W, _ = synth.weight(d_out, d_in, seed=4, k_outliers=cfg.k(d_in), device=gpu)
    layer = bsq.bsq_encode(cfg, codec, W)
    X = synth.activation(d_in, seed=6, device=gpu, batch=M)
    A, B = synth.lora(d_out, d_in, 16, seed=2, device=gpu)
    Y = bsq.bsq_gemm(cfg, codec, layer, X, lora=(A, B), y_dtype=torch.float32)
    rms = float(Y.square().mean().sqrt())
    for g0 in range(0, layer.row_groups, 37):
        g1 = min(g0 + 37, layer.row_groups)
        r0, r1 = 64 * g0, min(64 * g1, d_out)
        part = bsq.Layer(cfg, [c[g0:g1] for c in layer.codes], [g[g0:g1] for g in layer.gains], layer.idx,
                         layer.q8[r0:r1], layer.scale, r1 - r0, d_in, 1, layer.bits)
        Yp = bsq.bsq_gemm(cfg, codec, part, X, lora=(A, B[r0:r1].contiguous()), y_dtype=torch.float32)
        assert float((Y[:, r0:r1] - Yp).abs().max()) <= 1e-4 * rms, f"rows {r0}..{r1}"


@pytest.mark.parametrize("d", [8, 16])
def test_workspace_of_the_tiled_path_is_still_accepted(d, gpu):
    """A workspace too small for the decoded weights: the call is accepted and
    agrees with the other path to twice the rounding of a bf16 weight."""
    M, d_out, d_in = 1024, 300, 1024
    say(f"dense gemm small workspace d={d}")
    cfg = bsq.Config(d=d, hidden=d)
    codec = bsq.bsq_codec_prepare(cfg, decoders(cfg, seed=3), device=gpu)
    W, _ = synth.weight(d_out, d_in, seed=4, k_outliers=cfg.k(d_in), device=gpu)
    layer = bsq.bsq_encode(cfg, codec, W)
    X = synth.activation(d_in, seed=6, device=gpu, batch=M)
    Y = bsq.bsq_gemm(cfg, codec, layer, X, y_dtype=torch.float32)
    # the tiled path's scratch: T, X~ and X[:, idx] of padded tokens, no K splits or at most 8
    mp, kp = (M + 255) // 256 * 256, (d_in + 127) // 128 * 128
    small = 1024 + mp * (64 + 2 * kp + 2 * 32) + 8 * 4 * mp * 384
    need = bsq.bsq_workspace_bytes(cfg, bsq.OP_GEMM, 1, d_out, d_in, M)
    raw = torch.zeros(max(small, need) + 256, dtype=torch.uint8, device=gpu)
    ws = raw[(-raw.data_ptr()) % 256:]
    refused = 0
    for size in (need, need - 256, need // 2, mp * (64 + 2 * kp)):
        out = torch.full_like(Y, float("nan"))
        try:
            bsq.bsq_gemm(cfg, codec, layer, X, out=out, ws=ws[:size])
        except Exception as e:  # noqa: BLE001
            assert "small" in str(e).lower(), str(e)
            refused += 1
            continue
        # both paths round the same weights to bf16 and sum in fp32: they
        # differ by the order of d_in additions, far below 2^-16 of the rms
        assert float((out - Y).abs().max()) <= 2.0 ** -16 * float(Y.square().mean().sqrt()) * 16
    assert refused >= 1
