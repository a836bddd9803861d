"""The decode-once GEMM (many tokens) against the oracle, at the edges of its
tiles, for every (d, stages), payload format and output layout, with the
per-output bars of parity_bounds."""
import dataclasses

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


def planned_bytes(d_out, d_in, M, k, tile, ksplit):
    """The decode-once workspace for blocks of tile = (tokens, rows) and a K
    split: header, T, its partial sums, both operands and the split's fp32 tiles
    (one slab)."""
    up = lambda n, m: (n + m - 1) // m * m  # noqa: E731
    steps = (d_in + 127) // 128
    row = up(4 * steps + up(k, 32) // 32 + 2, 2) * 64
    mp, rows = up(M, tile[0]), up(d_out, tile[1])
    parts = ksplit * mp * rows * 4 if ksplit > 1 else 0
    return 256 + up(mp * 64, 256) * (1 + (steps + 3) // 4) + (mp + rows) * row + parts


def compare(M, d_out, d_in, kw, rank, gpu, ws_bytes=None):
    """Both output layouts against the oracle; the fp32 result."""
    say(f"gemm M={M} {d_out}x{d_in} {kw} rank={rank} workspace {ws_bytes or 'as reported'}")
    cfg = bsq.Config(**kw)
    oc = dataclasses.replace(ocfg(cfg), protect_axis=cfg.protect_axis)
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
    ws = None
    if ws_bytes:
        raw = torch.empty(ws_bytes + 256, dtype=torch.uint8, device=gpu)
        ws = raw[(-raw.data_ptr()) % 256:][:ws_bytes]
    Y = bsq.bsq_gemm(cfg, codec, layer, X, lora=lora, y_dtype=torch.float32, ws=ws)
    # bf16 rows of an odd pitch, and activations of a longer pitch, in one more call
    wide = torch.empty((M, d_out + 3), dtype=torch.bfloat16, device=gpu)[:, :d_out]
    Xw = torch.empty((M, d_in + 8), dtype=torch.bfloat16, device=gpu)[:, :d_in].copy_(X)
    Yb = bsq.bsq_gemm(cfg, codec, layer, Xw, lora=lora, out=wide, ws=ws)
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
    return Y


@pytest.mark.parametrize("M,d_out,d_in,kw,rank", CASES, ids=[f"{c[0]}x{c[1]}x{c[2]}-d{c[3]['d']}" for c in CASES])
def test_many_tokens_match_oracle(M, d_out, d_in, kw, rank, gpu):
    compare(M, d_out, d_in, kw, rank, gpu)


# K split over blocks of every tile (tokens x rows), ragged in both: (M, d_out,
# d_in, d, rank, tile, splits); the tile is the one the reported size stands for
SPLITS = [(1030, 260, 3000, 8, 16, (128, 128), 4), (400, 4100, 4000, 8, 16, (256, 128), 3),
          (900, 1300, 5008, 16, 0, (256, 128), 4), (800, 5000, 6000, 8, 5, (256, 192), 2),
          (900, 4100, 6000, 8, 0, (256, 256), 3)]


@pytest.mark.parametrize("M,d_out,d_in,d,rank,tile,splits", SPLITS, ids=["%dx%dx%d" % c[:3] for c in SPLITS])
def test_split_tiles_match_oracle(M, d_out, d_in, d, rank, tile, splits, gpu):
    cfg = bsq.Config(d=d, hidden=d)
    need = bsq.bsq_workspace_bytes(cfg, bsq.OP_GEMM, 1, d_out, d_in, M)
    assert need == planned_bytes(d_out, d_in, M, cfg.k(d_in), tile, splits), "another tile or split was planned"
    compare(M, d_out, d_in, dict(d=d, hidden=d), rank, gpu)


@pytest.mark.parametrize("rank", [0, 16])
@pytest.mark.parametrize("d", [8, 16])
def test_protected_rows_of_many_tokens_match_oracle(d, rank, gpu):
    """The decode-once product of the coded rows, then the protected rows from
    the T that it leaves in the workspace."""
    compare(1100, 200, 1008, dict(d=d, hidden=d, protect_axis=1, protect_num=1, protect_den=20), rank, gpu)


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


# (M, d_out, d_in, d): every tile of the tiled path that a reported workspace no
# longer leads to: 128 tokens x 128 rows and x 64 rows (d = 8), 256 x 64 and
# 128 x 128 (d = 16)
SMALL_WS = [(1040, 4100, 520, 8), (1030, 1090, 520, 8), (1030, 2500, 528, 16), (100, 1000, 384, 16)]


@pytest.mark.parametrize("stages", [1, 2, 3, 4])
@pytest.mark.parametrize("M,d_out,d_in,d", SMALL_WS, ids=["%dx%dx%d-d%d" % c for c in SMALL_WS])
def test_workspace_of_the_tiled_path_is_still_accepted(M, d_out, d_in, d, stages, gpu):
    """A workspace too small for the decoded weights: the smallest accepted size
    (by bisection) is below theirs, and its result, which decodes per token
    tile, matches the oracle as the other does. The two differ in the order of
    d_in fp32 additions, so some sums differ."""
    kw = dict(d=d, hidden=d, stages=stages)
    cfg = bsq.Config(**kw)
    need = bsq.bsq_workspace_bytes(cfg, bsq.OP_GEMM, 1, d_out, d_in, M)
    assert need > 2 * d_out * d_in, "the shape does not decode once"
    codec = bsq.bsq_codec_prepare(cfg, decoders(cfg, seed=3), device=gpu)
    layer = bsq.layer_empty(cfg, d_out, d_in, 1, gpu)
    for t in layer.codes + layer.gains + [layer.idx, layer.q8, layer.scale, layer.bits]:
        t.zero_()
    X = synth.activation(d_in, seed=6, device=gpu, batch=M)
    raw = torch.empty(need + 256, dtype=torch.uint8, device=gpu)
    ws = raw[(-raw.data_ptr()) % 256:]
    out = torch.empty((M, d_out), dtype=torch.float32, device=gpu)

    def accepted(size):
        try:
            bsq.bsq_gemm(cfg, codec, layer, X, out=out, ws=ws[:size])
        except bsq.BsqError as e:
            assert "too small" in str(e), str(e)
            return False
        return True

    lo, hi = 0, need  # refused, accepted
    while hi - lo > 256:
        mid = (lo + hi) // 512 * 256
        lo, hi = (lo, mid) if accepted(mid) else (mid, hi)
    torch.cuda.synchronize()
    assert hi < 2 * d_out * d_in + M * d_in * 2, "the smallest workspace has room for both operands"
    once = compare(M, d_out, d_in, kw, 16, gpu)
    tiled = compare(M, d_out, d_in, kw, 16, gpu, ws_bytes=hi)
    assert not torch.equal(once, tiled), "the small workspace did not change the path"


@pytest.mark.parametrize("stages", [1, 2, 3, 4])
def test_tiled_path_of_256_tokens_matches_oracle(stages, gpu):
    """128-token tiles of 128-row blocks at d = 8, which up to 256 tokens of few
    or long rows take with the reported workspace."""
    kw = dict(d=8, hidden=8, stages=stages)
    assert bsq.bsq_workspace_bytes(bsq.Config(**kw), bsq.OP_GEMM, 1, 4100, 4616, 200) < 2 * 4100 * 4616
    compare(200, 300, 4616, kw, 16, gpu)
    compare(200, 4100, 4616, kw, 0, gpu)
