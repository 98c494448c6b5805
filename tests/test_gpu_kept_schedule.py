"""A row schedule that serves several calls of a trajectory: the tickets are at zero again behind every call, all rows are
computed whatever the mask has become, and nothing of a result depends on the order of the rows.  Recorded calls, of any path:
what a replay gives depends on its inputs and on the mask as it stands then."""
import numpy as np
import pytest
import torch

from paper_2511_11062_amd import inputs
import parity

pytestmark = pytest.mark.gpu

STEPS = 11  # more than a schedule serves
# short rows that are drawn (one over a round of workgroups; some cut at an empty mask), too short to be drawn, long rows
SHAPES = [(27, 128 * 19 - 5, 0), (12, 128 * 110, 2), (25, 128 * 37, 0), (53, 128 * 13 - 60, 0), (3, 128 * 193 - 1, 1),
          (5, 128 * 200, 2)]


def trajectory(heads, tokens, flags, thresholds, fresh_schedules, q, k, v):
    """Outputs and masks of all steps; fresh_schedules: the mask is exported and imported before every call."""
    from paper_2511_11062_amd import lite_attn as la
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=len(thresholds), flags=flags)
    outs, masks = [], []
    try:
        la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
        for t, thr in enumerate(thresholds):
            if fresh_schedules and t > 0:
                la.lite_attn_mask_import(h, masks[-1], t)
            out = torch.full_like(q, float("nan"))
            s = t % 2  # two sets of inputs in turn, so that later steps mark too
            la.lite_attn_fwd(q[s:s + 1].data_ptr(), k[s:s + 1].data_ptr(), v[s:s + 1].data_ptr(), out[:1].data_ptr(), h, thr, t)
            torch.cuda.synchronize()
            outs.append(out[0].view(torch.int16).cpu())
            masks.append(la.lite_attn_mask_export(h).copy())
    finally:
        la.lite_attn_free_mask(h)
    return outs, masks


def layer(heads, tokens):
    wl = inputs.Workload("kept", 1, heads, (1, 1, tokens), steps=2, seed=17)
    seq = inputs.DriftSequence(wl, "cuda")
    steps = [next(seq) for _ in range(2)]
    return [torch.cat([s[x] for s in steps]) for x in range(3)]


@pytest.mark.parametrize("heads,tokens,flags", SHAPES)
def test_kept_schedule_gives_what_a_fresh_one_gives(heads, tokens, flags):
    path = parity.path_of(1, heads, tokens, flags)
    assert path.rows > 512
    q, k, v = layer(heads, tokens)
    thresholds = [-1.5] * 5 + [-0.8] + [-1.5] * (STEPS - 6)  # one looser call on the way: the schedule is made again
    outs, masks = trajectory(heads, tokens, flags, thresholds, False, q, k, v)
    ref_outs, ref_masks = trajectory(heads, tokens, flags, thresholds, True, q, k, v)
    assert np.unpackbits(masks[-1].view(np.uint8)).sum() > np.unpackbits(masks[0].view(np.uint8)).sum() > 0
    for t in range(STEPS):
        assert np.array_equal(masks[t], ref_masks[t]), t
        assert torch.equal(outs[t], ref_outs[t]), t


@pytest.mark.parametrize("heads,tokens", [(12, 128 * 110), (18, 128 * 29)])
def test_cut_rows_while_a_kept_schedule_says_that_the_mask_is_empty(heads, tokens):
    """Calls whose threshold marks nothing, then one that does: the schedule made in between was made for an empty mask."""
    assert parity.path_of(1, heads, tokens).rows > 512 and parity.path_of(1, heads, tokens).rows % 512 <= 320
    q, k, v = layer(heads, tokens)
    thresholds = [-60.0, -60.0, -60.0, -1.5, -1.5, -1.5]
    outs, masks = trajectory(heads, tokens, 0, thresholds, False, q, k, v)
    ref_outs, ref_masks = trajectory(heads, tokens, 0, thresholds, True, q, k, v)
    assert not masks[2].any() and masks[3].any()
    for t in range(len(thresholds)):
        assert np.array_equal(masks[t], ref_masks[t]) and torch.equal(outs[t], ref_outs[t]), t


@pytest.mark.parametrize("heads,tokens", [(12, 128 * 110), (18, 128 * 29)])
def test_cut_rows_where_an_empty_mask_was_imported(heads, tokens):
    """Steps whose counters tell of marks that an import has taken back: the rows are cut as where no call has marked."""
    from paper_2511_11062_amd import lite_attn as la
    assert parity.path_of(1, heads, tokens).rows % 512 in range(1, 321)
    q, k, v = layer(heads, tokens)
    out = torch.full((2,) + tuple(q.shape[1:]), float("nan"), dtype=q.dtype, device="cuda")
    masks = []
    for x, steps in enumerate(([(-1.5, 0), (-1.5, 1), None, (-60.0, 1), (-1.5, 2)],
                               [(-60.0, 0), (-60.0, 1), None, (-60.0, 1), (-1.5, 2)])):
        h = la.lite_attn_init_mask(1, heads, tokens, max_steps=3)
        try:
            la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
            for step in steps:
                if step is None:
                    la.lite_attn_mask_import(h, np.zeros(la.lite_attn_mask_words(h), dtype=np.uint64), 1)
                else:
                    la.lite_attn_fwd(q[:1].data_ptr(), k[:1].data_ptr(), v[:1].data_ptr(), out[x:].data_ptr(), h, *step)
            torch.cuda.synchronize()
            masks.append(la.lite_attn_mask_export(h))
        finally:
            la.lite_attn_free_mask(h)
    assert masks[0].any() and np.array_equal(masks[0], masks[1])
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))


@pytest.mark.parametrize("heads,tokens,flags", SHAPES[1:4])
def test_kept_schedule_in_a_graph(heads, tokens, flags):
    """Four steps recorded at once, the last two on the second's schedule, replayed with eager work between the replays."""
    from paper_2511_11062_amd import lite_attn as la
    q, k, v = layer(heads, tokens)
    thresholds = [-1.5] * 4
    ref, ref_masks = trajectory(heads, tokens, flags, thresholds, False, q, k, v)
    out = torch.empty((4,) + tuple(q.shape[1:]), dtype=q.dtype, device="cuda")
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=4, flags=flags)
    side = torch.cuda.Stream()
    try:
        la.lite_attn_set_stream(h, side.cuda_stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for t, thr in enumerate(thresholds):
                s = t % 2
                la.lite_attn_fwd(q[s:s + 1].data_ptr(), k[s:s + 1].data_ptr(), v[s:s + 1].data_ptr(),
                                 out[t:t + 1].data_ptr(), h, thr, t)
        for _ in range(3):
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for t in range(4):
                assert torch.equal(out[t].view(torch.int16).cpu(), ref[t]), t
            assert np.array_equal(la.lite_attn_mask_export(h), ref_masks[-1])
        # and an eager call behind the replays
        la.lite_attn_fwd(q[:1].data_ptr(), k[:1].data_ptr(), v[:1].data_ptr(), out[:1].data_ptr(), h, thresholds[0], 0)
        torch.cuda.synchronize()
        assert torch.equal(out[0].view(torch.int16).cpu(), ref[0])
    finally:
        la.lite_attn_free_mask(h)


# (short rows of every kind, rows with lists, few rows in pieces and in segments)
@pytest.mark.parametrize("heads,tokens,flags", SHAPES + [(18, 128 * 29, 3), (5, 128 * 31, 0), (2, 128 * 16, 2)])
def test_later_call_recorded_alone(heads, tokens, flags):
    """Step 2 by itself in a graph, replayed between calls of which the host knew nothing when it was recorded: output and
    mask, bit for bit, are those of an eager call on a handle that has imported the mask."""
    from paper_2511_11062_amd import lite_attn as la
    q, k, v = layer(heads, tokens)
    path = parity.path_of(1, heads, tokens, flags)
    dense, marking = -float("inf"), -1.5
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=4, flags=flags)
    eager = la.lite_attn_init_mask(1, heads, tokens, max_steps=4, flags=flags)
    out, ref = torch.empty_like(q), torch.empty_like(q)
    side = torch.cuda.Stream()

    def call(handle, o, threshold, step, s):
        la.lite_attn_fwd(q[s:s + 1].data_ptr(), k[s:s + 1].data_ptr(), v[s:s + 1].data_ptr(), o[:1].data_ptr(), handle,
                         threshold, step)

    def check(what, run, step, s):
        mask = la.lite_attn_mask_export(h)
        la.lite_attn_mask_import(eager, mask, step)
        ref.fill_(float("nan"))
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        call(eager, ref, marking, step, s)
        run()
        torch.cuda.synchronize()
        assert torch.equal(out[0].view(torch.int16), ref[0].view(torch.int16)), what
        assert np.array_equal(la.lite_attn_mask_export(h), la.lite_attn_mask_export(eager)), what

    try:
        la.lite_attn_set_stream(h, side.cuda_stream)
        la.lite_attn_set_stream(eager, side.cuda_stream)
        torch.cuda.synchronize()
        for t in (0, 1):
            call(h, out, marking, t, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(h, out, marking, 2, 1)
        check("as it was recorded", graph.replay, 2, 1)
        for t in (0, 1):
            call(h, out, dense, t, 0)
        check("behind dense calls", graph.replay, 2, 1)
        if path.rows > 512:  # (few rows are cut by the live tiles that step 1 has counted)
            call(h, out, dense, 0, 0)
            check("behind step 0", graph.replay, 2, 1)
            check("again", graph.replay, 2, 1)
        rng = np.random.default_rng(3)
        for share in (0.0, 0.5):
            tiles = rng.random((path.rows, path.Tk)) < share
            la.lite_attn_mask_import(h, parity.pack_mask(tiles.astype(np.uint8)).ravel(), 2)
            check("imported, %g" % share, graph.replay, 2, 1)
        call(h, out, dense, 0, 0)
        graph.replay()
        torch.cuda.synchronize()
        check("eager behind a replay", lambda: call(h, out, marking, 1, 0), 1, 0)
    finally:
        la.lite_attn_free_mask(h)
        la.lite_attn_free_mask(eager)
