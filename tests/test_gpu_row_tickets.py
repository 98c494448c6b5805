"""Rows beyond the first round of workgroups are drawn from counters, one per XCD, and by whichever XCD runs dry first: every
row is computed once, call after call, whatever the lengths of the eight lists."""
import numpy as np
import pytest
import torch

import parity

pytestmark = pytest.mark.gpu


# one row beyond the few; lists a row longer than the first round, and of unequal lengths; an XCD (or four) without any chunk of
# rows, with one that is not full; more rows than are scheduled (their last chunks have places without rows); rows too short to
# be drawn, which go by place (up to 15 tiles)
@pytest.mark.parametrize("heads,tiles", [(513, 1), (521, 1), (27, 19), (40, 64), (3, 193), (1, 600), (9, 200), (33001, 1),
                                         (4681, 7), (2053, 16)])
def test_every_row_once_call_after_call(heads, tiles):
    """Scores of zero: a row's output is the mean of the values of its live tiles, each of them one number.  The counters of a
    call add up over its rows, so a row computed twice, or not at all, shows there too."""
    from paper_2511_11062_amd import lite_attn as la
    n, steps = 128 * tiles, 3
    assert parity.path_of(1, heads, n).rows > 512
    rng = np.random.default_rng(heads + tiles)
    value = rng.integers(-8, 9, size=(heads, tiles)).astype(np.float32)
    q = torch.zeros(1, heads, n, 128, dtype=torch.bfloat16, device="cuda")
    v = torch.from_numpy(value).cuda().repeat_interleave(128, 1)[None, :, :, None].expand(-1, -1, -1, 128).to(torch.bfloat16)
    v = v.contiguous()
    h = la.lite_attn_init_mask(1, heads, n, max_steps=steps + 1)
    la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
    try:
        for t in range(steps):
            live = rng.random((heads, tiles, tiles)) < rng.random((heads, 1, 1)) if t else np.ones((heads, tiles, tiles), bool)
            if t:
                la.lite_attn_mask_import(h, parity.pack_mask((~live).astype(np.uint8)), t)
            out = torch.full_like(q, float("nan"))
            la.lite_attn_fwd(q.data_ptr(), q.data_ptr(), v.data_ptr(), out.data_ptr(), h, -float("inf"), t)
            st = la.lite_attn_skip_stats(h, t)
            assert st.tiles_skipped_in == int((~live).sum())
            count = live.sum(axis=2)
            want = np.einsum("hij,hj->hi", live.astype(np.float32), value) / np.maximum(count, 1)
            got = out.view(heads, tiles, 128, 128).float()
            ref = torch.from_numpy(want).cuda()[:, :, None, None]
            # weights of 1 are exact, the sum is of integers: one rounding of the quotient and one to bf16
            assert (got - ref).abs().max().item() <= 8 * 2.0 ** -8
    finally:
        la.lite_attn_free_mask(h)
