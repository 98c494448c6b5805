"""Calls with few Q-tile rows: rows cut into segments (one workgroup each) whose partial results a second kernel merges,
and rows kept whole, both finding their tiles from the mask row itself.  Sizes at which that can go wrong: one tile, fewer
live tiles than segments, segment lengths with a remainder, mask rows of one, exactly one and more than one 64-bit word,
the last size with few rows and the first without."""
import numpy as np
import pytest
import torch

from paper_2511_11062_amd import inputs
import parity

pytestmark = pytest.mark.gpu


def layer(heads, tokens, text=0, batch=1, seed=71):
    return inputs.Workload("few", batch, heads, (1, 1, tokens - text), text_tokens=text, steps=3, seed=seed)


@pytest.mark.parametrize("diagonal_first", [False, True])
@pytest.mark.parametrize("heads,tokens,text", [(1, 128 * 5 - 1, 0), (2, 128 * 17 + 3, 40), (1, 128 * 63 + 5, 0),
                                               (1, 128 * 64, 0), (1, 128 * 65 + 7, 130), (7, 128 * 9 + 64, 0)])
def test_marking_across_segments(heads, tokens, text, diagonal_first):
    """Three steps against the oracle, deferred marking: the tiles of a later segment are judged against the maximum
    carried over from the earlier ones; then with the literal PV skip, whose rows stay whole."""
    thr = [-3.0, -1.5, -0.7]
    reps = parity.run_sequence_check(layer(heads, tokens, text), steps=3, thresholds=thr, diagonal_first=diagonal_first)
    assert reps[-1]["skipped_out"] > 0.02
    parity.run_sequence_check(layer(heads, tokens, text), steps=2, thresholds=thr, diagonal_first=diagonal_first,
                              immediate=True)


@pytest.mark.parametrize("flags", [0, 1, 2, 3])
@pytest.mark.parametrize("batch,heads,tokens,text", [(2, 12, 128 * 37 - 51, 0), (1, 8, 128 * 65 + 7, 130),
                                                     (1, 5, 128 * 128, 0), (1, 3, 128 * 192 - 1, 0)])
def test_marking_beyond_one_round_of_workgroups(batch, heads, tokens, text, flags):
    """More rows than run side by side, at most 192 tiles a row: a step 0 without a schedule, whose marks the scheduled steps
    read (one to three mask words a row), thresholds that rise, protected text, either order, deferred and literal PV skip;
    sampled rows against the oracle.  Then the trajectory on its own: the counters of every step against the masks."""
    from paper_2511_11062_amd import lite_attn as la
    wl = layer(heads, tokens, text, batch=batch)
    path = parity.path_of(batch, heads, tokens, flags)
    assert path.nseg == 1 and 512 < path.rows <= 32768
    thr = [-3.0, -1.5, -0.7]
    reps = parity.run_sequence_check(wl, steps=3, thresholds=thr, sample_rows=16, seed=flags, immediate=bool(flags & 1),
                                     diagonal_first=bool(flags & 2))
    assert reps[-1]["skipped_out"] > 0.02
    seq = inputs.DriftSequence(wl, "cuda:0")
    h = la.lite_attn_init_mask(batch, heads, tokens, protect=wl.protect, max_steps=3, flags=flags)
    try:
        la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
        before = np.zeros((path.rows, path.Tk), dtype=bool)
        for t in range(3):
            q, k, v = (x.contiguous() for x in next(seq))
            out = torch.full_like(q, float("nan"))
            la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, thr[t], t)
            st = la.lite_attn_skip_stats(h, t)
            after = parity.unpack_mask(la.lite_attn_mask_export(h).reshape(path.rows, path.W), path.Tk) != 0
            assert torch.isfinite(out).all() and not (before & ~after).any()
            assert st.tiles_skipped_in == int(before.sum()) and st.tiles_newly_marked == int((after & ~before).sum())
            # entries of the list the row would have: maximal runs of live tiles, a wrap-around run counted twice
            starts = ~before & np.pad(before, ((0, 0), (1, 0)), constant_values=True)[:, :-1]
            runs = int(starts.sum())
            if flags & 2:                                       # diagonal first: a run across the diagonal is cut there
                i = np.tile(np.arange(path.Tq), path.BH)
                r = np.arange(path.rows)
                runs += int((~before[r, i] & ~before[r, np.maximum(i - 1, 0)] & (i > 0)).sum())
            assert st.live_list_bytes == 4 * runs
            before = after
        assert before.any()
    finally:
        la.lite_attn_free_mask(h)


@pytest.mark.parametrize("heads,tiles", [(1, 5), (2, 16), (1, 65), (3, 100), (4, 128), (1, 513), (27, 19),
                                         (3, 192), (8, 193), (520, 2), (33000, 1), (3301, 10)])
@pytest.mark.parametrize("live", [0.02, 0.5, "uneven"])
def test_every_row_under_sparse_masks(heads, tiles, live):
    """Random imported masks, many rows with fewer live tiles than segments and some with none, every row against
    block-masked softmax attention in fp32; 512 and 513 rows, 192 and 193 tiles a row and 32768 rows are where the path changes
    (no schedule / rows scheduled / lists and V^T; beyond 32768 rows, chunks of rows dealt in turn)."""
    from paper_2511_11062_amd import lite_attn as la
    n = 128 * tiles - 3
    g = torch.Generator(device="cuda").manual_seed(1000 * heads + tiles)
    q, k, v = (torch.randn(1, heads, n, 128, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    rng = np.random.default_rng(tiles)
    # "uneven": a few heads hold nearly all live tiles, so that an XCD's equal share of the work is most of the rows
    share = np.where(np.arange(heads)[:, None, None] < max(1, heads // 8), 1.0, 0.01) if live == "uneven" else live
    skip = rng.random((heads, tiles, tiles)) >= share
    h = la.lite_attn_init_mask(1, heads, n, max_steps=2)
    out = torch.full_like(q, float("nan"))
    try:
        la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
        la.lite_attn_mask_import(h, parity.pack_mask(skip.astype(np.uint8)), 1)
        la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, -float("inf"), 1)
        st = la.lite_attn_skip_stats(h, 1)
        bits = la.lite_attn_mask_export(h)
    finally:
        la.lite_attn_free_mask(h)
    assert st.tiles_skipped_in == int(skip.sum()) and st.tiles_newly_marked == 0
    assert st.live_list_bytes == 4 * int((~skip & np.pad(skip, ((0, 0), (0, 0), (1, 0)), constant_values=True)[..., :-1]).sum())
    assert np.array_equal(bits, parity.pack_mask(skip.astype(np.uint8)).ravel())
    dead = torch.from_numpy(skip).cuda()
    for x in range(heads) if heads < 1000 else list(range(0, heads, 997)) + [heads - 1]:
        kf, vf = k[0, x].float().t().contiguous(), v[0, x].float()
        for i0 in range(0, tiles, 32):
            r0, r1 = 128 * i0, min(n, 128 * (i0 + 32))
            s = (q[0, x, r0:r1].float() @ kf) * 128 ** -0.5
            cols = dead[x, i0:i0 + 32].repeat_interleave(128, 0)[:r1 - r0].repeat_interleave(128, 1)[:, :n]
            ref = torch.nan_to_num(torch.softmax(s.masked_fill_(cols, -float("inf")), dim=1), nan=0.0) @ vf
            d = (out[0, x, r0:r1].float() - ref).abs()
            assert torch.isfinite(out[0, x, r0:r1]).all()
            # weights and result are rounded to bf16 (2^-9 each) of values up to max|O|
            assert d.max().item() <= 1e-2 * ref.abs().max().clamp(min=1e-3).item(), (x, i0)


@pytest.mark.parametrize("diagonal_first", [False, True])
@pytest.mark.parametrize("batch,heads,tokens,text", [(1, 1, 128 * 5 - 60, 0), (2, 1, 128 * 6, 0), (1, 1, 128 * 7, 0),
                                                     (1, 1, 128 * 33 + 1, 0), (1, 1, 128 * 49, 200), (3, 1, 128 * 17, 0)])
def test_marking_in_quarters(batch, heads, tokens, text, diagonal_first):
    """The merge pass judges a short row's tiles in quarters of its places, whatever the segments were: quarters
    with a remainder or empty, batch entries; masks and outputs of three steps against the oracle."""
    assert parity.path_of(batch, heads, tokens).nseg > 1
    parity.run_sequence_check(layer(heads, tokens, text, batch), steps=3, thresholds=[-2.0, -1.0, -0.4],
                              diagonal_first=diagonal_first)
