"""The GEMM's choice of path and tiles, seen from the workspace it asks for
(host only)."""
import pytest

import paper_2607_08643_amd as bsq


def gemm_ws(cfg, d_out, d_in, M):
    return bsq.bsq_workspace_bytes(cfg, bsq.OP_GEMM, 1, d_out, d_in, M)


@pytest.mark.parametrize("d_out,d_in,M,full", [(2048, 8192, 257, 384), (8192, 8192, 257, 384), (6144, 4096, 129, 256)])
def test_padded_tokens_count_in_the_choice_of_tiles(d_out, d_in, M, full):
    """A ragged last tile is written as a whole one, so M tokens take no more
    scratch than the tokens that fill the same tiles (257 used to take tiles of
    512 tokens in twice the splits)."""
    cfg = bsq.Config(d=8, hidden=8)
    assert gemm_ws(cfg, d_out, d_in, M) <= gemm_ws(cfg, d_out, d_in, full)


# (d, stages, d_out, d_in, M, decode-once): cells where both paths were measured
# (replayed graphs, rotated layers) and one is faster by 5% or more with and
# without an adapter
MEASURED = [
    (8, 2, 12288, 4096, 264, True), (8, 2, 12288, 4096, 2000, True), (8, 2, 4096, 4096, 160, True),
    (8, 1, 18944, 3584, 256, True), (8, 4, 25600, 5120, 256, True), (8, 2, 4096, 12288, 512, True),
    (8, 1, 64, 256, 257, True), (8, 2, 20480, 5120, 192, True),
    (8, 1, 16384, 8192, 256, False), (8, 2, 16384, 8192, 129, False), (8, 2, 8192, 8192, 192, False),
    (8, 1, 28672, 8192, 256, False), (8, 1, 25600, 5120, 160, False), (8, 1, 5120, 25600, 257, False),
    (8, 2, 5120, 25600, 320, False),
    (16, 2, 1024, 4096, 65, True), (16, 2, 12288, 4096, 256, True), (16, 1, 64, 4096, 96, True),
    (16, 4, 1024, 16384, 128, True), (16, 2, 25600, 5120, 160, True), (16, 1, 12288, 256, 65, True),
    (16, 1, 4096, 12288, 65, False), (16, 1, 12288, 4096, 128, False), (16, 1, 5120, 25600, 96, False),
    (16, 3, 4096, 12288, 96, False), (16, 2, 5120, 25600, 128, False), (16, 3, 8192, 4096, 65, False),
    (16, 1, 151936, 1024, 65, False),
]


@pytest.mark.parametrize("d,stages,d_out,d_in,M,once", MEASURED, ids=["d%d-s%d-%dx%d-M%d" % c[:5] for c in MEASURED])
def test_the_measured_faster_path_is_taken(d, stages, d_out, d_in, M, once):
    """Room for the decoded bf16 weights is asked for where decoding them once
    measured faster, and only there (the tiled path's own scratch is far
    smaller than the weights in the cells where it won)."""
    cfg = bsq.Config(d=d, stages=stages, hidden=d)
    assert (gemm_ws(cfg, d_out, d_in, M) >= 2 * d_out * d_in) == once
