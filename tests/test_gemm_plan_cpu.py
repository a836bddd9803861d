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
