"""Step 0 of calls with few rows clears the counters inside the attention launch and keeps its own marks per row: what the
statistics say must not depend on what the handle counted before."""
import numpy as np
import pytest
import torch

import parity
from paper_2511_11062_amd import inputs

pytestmark = pytest.mark.gpu


# whole rows, rows cut into segments, pairs; mask rows of one, two and three words; the most rows there are
@pytest.mark.parametrize("heads,tokens", [(3, 85), (2, 128 * 16), (5, 3913), (3, 128 * 65 - 4), (2, 128 * 130), (128, 500)])
@pytest.mark.parametrize("flags", [0, 1, 2])
def test_second_trajectory_counts_like_the_first(heads, tokens, flags):
    from paper_2511_11062_amd import lite_attn as la
    path = parity.path_of(1, heads, tokens, flags)
    assert path.rows <= 512
    wl = inputs.Workload("counters", 1, heads, (1, 1, tokens), steps=3, seed=11)
    seq = inputs.DriftSequence(wl, "cuda:0")
    data = [tuple(x.contiguous() for x in next(seq)) for _ in range(3)]
    out = torch.empty_like(data[0][0])
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=3, flags=flags)
    la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
    seen = []
    try:
        for trajectory in range(2):
            skipped, stats = 0, []
            for t, (q, k, v) in enumerate(data):
                la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, [-2.0, -1.0, -0.3][t], t)
                st = la.lite_attn_skip_stats(h, t)
                mask = parity.unpack_mask(la.lite_attn_mask_export(h).reshape(path.rows, path.W), path.Tk)
                assert st.tiles_skipped_in == skipped and st.tiles_newly_marked == int(mask.sum()) - skipped
                skipped = int(mask.sum())
                stats.append((st.tiles_newly_marked, st.live_list_bytes))
            assert stats[0][1] == 4 * path.rows * 1 + (4 * heads * (path.Tq - 1) if flags & 2 else 0)
            seen.append(stats)
        assert seen[0] == seen[1]
        assert [la.lite_attn_skip_stats(h, t).tiles_newly_marked for t in range(3)] == [s[0] for s in seen[0]]
        if path.Tk > 4:
            assert skipped > 0
    finally:
        la.lite_attn_free_mask(h)


@pytest.mark.parametrize("heads,tokens,max_steps", [(2, 300, 700), (1, 128 * 16, 700), (1, 200, 1 << 20)])
def test_counters_of_many_steps(heads, tokens, max_steps):
    """More counters than a workgroup has threads: every step of a second trajectory counts as in the first."""
    from paper_2511_11062_amd import lite_attn as la
    steps = 700                                                # (2^20: cleared by a launch)
    path = parity.path_of(1, heads, tokens)
    wl = inputs.Workload("counters", 1, heads, (1, 1, tokens), steps=1, seed=12)
    q, k, v = (x.to("cuda:0").contiguous() for x in next(inputs.DriftSequence(wl, "cuda:0")))
    out = torch.empty_like(q)
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=max_steps)
    la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
    try:
        for trajectory in range(2):
            for t in range(steps):
                la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, -0.5, t)
            stats = [la.lite_attn_skip_stats(h, t) for t in range(steps)]
            marked = stats[0].tiles_newly_marked
            assert all(st.tiles_skipped_in == marked and st.tiles_newly_marked == 0 for st in stats[1:])
            assert len({st.live_list_bytes for st in stats[1:]}) == 1 and stats[0].live_list_bytes == 4 * path.rows
    finally:
        la.lite_attn_free_mask(h)
