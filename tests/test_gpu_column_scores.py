"""Column scores on both sides of the bound between their two kernels (a
workgroup per 64 columns in turns, a lane per column): the same bits."""
import numpy as np
import pytest
import torch

import paper_2607_08643_amd as bsq
from parity_bounds import say

pytestmark = pytest.mark.gpu


# 64-column groups at and just past 256 (under 64 rows), 768 and 1024 (under
# 512 rows of bf16, 256 of fp32), 1280 and 1536; fp32 with its seventh round of
# 256 just three quarters full and just not
@pytest.mark.parametrize("rows,groups,dtype", [(56, 256, torch.bfloat16), (56, 257, torch.bfloat16),
                                               (104, 768, torch.bfloat16), (104, 769, torch.bfloat16),
                                               (104, 1024, torch.float32), (104, 1025, torch.float32),
                                               (520, 1280, torch.bfloat16), (520, 1281, torch.bfloat16),
                                               (264, 1536, torch.float32), (264, 1537, torch.float32),
                                               (520, 1728, torch.float32), (520, 1727, torch.float32)])
def test_column_scores_at_the_bound_of_the_turns(rows, groups, dtype, gpu):
    """Scores of a down matrix alone (zero gate and up): the square roots of the
    sequential fp64 sums of squares, bit for bit."""
    say(f"column scores {rows} rows, {groups} groups, {dtype}")
    cols = 64 * groups
    g = torch.Generator(device=gpu).manual_seed(rows + groups)
    W = torch.randn((rows, cols), generator=g, device=gpu).to(dtype)
    Z = torch.zeros((cols, rows), dtype=dtype, device=gpu)
    _, sc = bsq.bsq_coupled_select(bsq.Config(d=8, hidden=8), Z, Z, W, with_scores=True)
    w = W.double().cpu().numpy()
    s = np.zeros(cols)
    for i in range(rows):
        s = s + w[i] * w[i]
    assert np.array_equal(sc.cpu().numpy().view(np.int64), np.sqrt(s).view(np.int64))
