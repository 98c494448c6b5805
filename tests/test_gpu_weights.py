"""The weights' reference is the running row maximum: a row's largest weight is exactly 1, whatever it met before."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def two_term_cancellation(heads, tiles):
    """q, k, v [1,heads,128*tiles,128] whose attention output is 0 if, and only if, the weights 1 and 0.75 come out exact.

    Score of key j for every query: 0 for one key and ln 0.75 for another, both in tile 1 (weights 1 and 0.75, which bf16
    holds exactly; values 3 and -4: 3 * 1 - 4 * 0.75 = 0); per query 0.2 to 5.4 below the top for two keys of tile 0, one in
    each column half (values 0); -30 everywhere else (values 0).  A reference left behind at the maximum of tile 0 makes the two
    weights 2^f and 0.75 * 2^f, which bf16 rounds with errors of their own: 3 * 2^-9 of the row sum survives."""
    n = 128 * tiles
    s = math.sqrt(128.0)
    q = torch.zeros(1, heads, n, 128, dtype=torch.float64)
    k = torch.zeros_like(q)
    v = torch.zeros_like(q)
    q[..., 0] = q[..., 1] = s / 8                          # features 0 and 1: a score in two bf16 pieces
    q[..., :2] = q[..., :2].bfloat16().double()
    q[..., 2] = -torch.linspace(0.2, 5.4, 128, dtype=torch.float64).repeat(tiles) * s   # feature 2: the keys of tile 0
    a = q[0, 0, 0, 0].item()
    k[..., 0] = -30.0 * s / a
    k[:, :, [3, 67], :2], k[:, :, [3, 67], 2] = 0.0, 1.0
    k[:, :, 128 + 70, 0] = 0.0
    x = math.log(0.75) * s / a
    hi = torch.tensor(x).bfloat16().item()
    k[:, :, 128 + 72, 0], k[:, :, 128 + 72, 1] = hi, x - hi
    v[:, :, 128 + 70], v[:, :, 128 + 72] = 3.0, -4.0
    return [t.to(torch.bfloat16).cuda() for t in (q, k, v)]


# rows cut into segments (two sizes), whole rows on pairs of wave groups, more rows than fit at once with one and with
# several tiles' lists to walk, rows with Skip-Lists and V^T
@pytest.mark.parametrize("heads,tiles", [(2, 16), (4, 64), (5, 31), (16, 32), (27, 19), (3, 193)])
@pytest.mark.parametrize("immediate", [False, True])
def test_largest_weight_is_exact(heads, tiles, immediate):
    from paper_2511_11062_amd import lite_attn as la
    q, k, v = two_term_cancellation(heads, tiles)
    out = torch.full_like(q, float("nan"))
    h = la.lite_attn_init_mask(1, heads, 128 * tiles, flags=la.LITE_ATTN_PV_SKIP_IMMEDIATE if immediate else 0)
    try:
        la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
        la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, -float("inf"), 0)
        torch.cuda.synchronize()
    finally:
        la.lite_attn_free_mask(h)
    # both weights lie 2^-9 (relative) inside their bf16 rounding interval, the scores and exponentials are off by some 2^-16:
    # the cancellation is exact
    worst = out.float().abs().max().item()
    assert worst <= 2.0 ** -20
