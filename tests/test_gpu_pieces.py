"""Few rows under a mask: rows cut into pieces by their live tiles, merged and judged by the piece that arrives last.  Sizes at
which that can go wrong: pairs and single groups; rows with no, one and all tiles; mask rows of one, exactly one and several
words; a ragged last tile; protected rows; the most rows that are cut."""
import ctypes

import numpy as np
import pytest
import torch

import parity
from paper_2511_11062_amd import inputs

pytestmark = pytest.mark.gpu


class Path(ctypes.Structure):                              # la::Geometry, whole
    _fields_ = [("Tq", ctypes.c_int), ("Tk", ctypes.c_int), ("W", ctypes.c_int), ("run_stride", ctypes.c_int),
                ("BH", ctypes.c_int), ("pieces", ctypes.c_int), ("rows", ctypes.c_int64), ("chunks", ctypes.c_int),
                ("pair", ctypes.c_int), ("nseg", ctypes.c_int), ("per_xcd", ctypes.c_int)]


def path_of(heads, tokens, flags=0, protect=(0, 0)):
    from paper_2511_11062_amd import lite_attn as la
    f = la._lib._ZN2la8geometryERK16lite_attn_desc_t
    old = f.restype, f.argtypes
    f.restype, f.argtypes = Path, [ctypes.POINTER(la.Desc)]
    p = f(ctypes.byref(la.make_desc(1, heads, tokens, flags=flags, protect=protect)))
    f.restype, f.argtypes = old
    return p


def layer(heads, tokens, text):
    return inputs.Workload("pieces", 1, heads, (1, 1, tokens - text), text_tokens=text, steps=3, seed=91)


SHAPES = [(9, 128 * 15, 0, 256), (5, 128 * 31 - 55, 100, 256), (10, 128 * 29 + 1, 0, 512), (30, 128 * 10, 33, 512),
          (4, 128 * 25, 0, 256), (2, 128 * 64, 0, 256), (2, 128 * 65 - 3, 200, 256), (1, 128 * 129 + 7, 0, 256),
          (5, 128 * 60 + 9, 0, 512), (17, 128 * 21, 0, 512)]


@pytest.mark.parametrize("diagonal_first", [False, True])
@pytest.mark.parametrize("heads,tokens,text,pieces", SHAPES)
def test_marking_across_pieces(heads, tokens, text, pieces, diagonal_first):
    """Three steps with rising thresholds against the oracle: outputs, and the tiles of a later piece judged against the maximum
    carried over from the earlier ones."""
    wl = layer(heads, tokens, text)
    assert path_of(heads, tokens, 2 * diagonal_first, wl.protect).pieces == pieces
    reps = parity.run_sequence_check(wl, steps=3, thresholds=[-2.0, -1.2, -0.6], diagonal_first=diagonal_first, sample_rows=40)
    assert reps[-1]["skipped_out"] > 0.02


@pytest.mark.parametrize("heads,tokens,text", [(5, 128 * 31 - 55, 100), (8, 128 * 20, 300)])
def test_protected_rows_of_the_literal_skip(heads, tokens, text):
    wl = layer(heads, tokens, text)
    assert path_of(heads, tokens, 3, wl.protect).pieces > 0 and path_of(heads, tokens, 1, wl.protect).pieces == 0
    parity.run_sequence_check(wl, steps=3, thresholds=[-2.0, -1.2, -0.6], diagonal_first=True, immediate=True, sample_rows=30)


@pytest.mark.parametrize("heads,tokens,pieces", [(9, 128 * 15 - 3, 256), (10, 128 * 29, 512), (2, 128 * 65 - 3, 256),
                                                 (5, 128 * 60, 512), (1, 128 * 170 - 1, 256), (2, 128 * 179, 512)])
def test_uneven_masks_handle_and_static(heads, tokens, pieces):
    """Imported masks with rows of every length, one without a live tile, one with all: every row against block-masked softmax in
    fp32; twice with the same result, bit for bit, whatever piece arrived last; then the allocation-free entry point's."""
    from paper_2511_11062_amd import lite_attn as la
    tiles, W = -(-tokens // 128), -(-tokens // 128 // 64)
    assert path_of(heads, tokens).pieces == pieces
    rng = np.random.default_rng(tokens)
    skip = rng.random((heads, tiles, tiles)) >= rng.random((heads, tiles, 1)) ** 2
    skip[0, 0] = True
    skip[-1, -1] = False
    skip[0, 1, 1:], skip[0, 1, 0] = True, False
    g = torch.Generator(device="cuda").manual_seed(tokens)
    q, k, v = (torch.randn(1, heads, tokens, 128, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    stream = torch.cuda.current_stream().cuda_stream
    packed = parity.pack_mask(skip.astype(np.uint8))
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=2)
    la.lite_attn_set_stream(h, stream)
    outs = []
    try:
        for _ in range(2):
            out = torch.full_like(q, float("nan"))
            la.lite_attn_mask_import(h, packed, 1)
            la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, -100.0, 1)   # (marks nothing)
            st = la.lite_attn_skip_stats(h, 1)
            assert np.array_equal(la.lite_attn_mask_export(h), packed.ravel())
            outs.append(out)
        # the counters of a step add up over its calls
        assert st.tiles_skipped_in == 2 * int(skip.sum()) and st.tiles_newly_marked == 0
    finally:
        la.lite_attn_free_mask(h)
    desc = la.make_desc(1, heads, tokens, max_steps=1)
    mask = torch.from_numpy(packed.ravel().view(np.int64).copy()).cuda()
    out = torch.full_like(q, float("nan"))
    la.lite_attn_fwd_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), desc, mask.data_ptr(), -100.0, stream)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], out)
    assert np.array_equal(mask.cpu().numpy().view(np.uint64), packed.ravel())
    dead = torch.from_numpy(skip).cuda()
    for x in range(heads):
        kf, vf = k[0, x].float().t().contiguous(), v[0, x].float()
        for i0 in range(0, tiles, 32):
            r0, r1 = 128 * i0, min(tokens, 128 * (i0 + 32))
            s = (q[0, x, r0:r1].float() @ kf) * 128 ** -0.5
            cols = dead[x, i0:i0 + 32].repeat_interleave(128, 0)[:r1 - r0].repeat_interleave(128, 1)[:, :tokens]
            ref = torch.nan_to_num(torch.softmax(s.masked_fill_(cols, -float("inf")), dim=1), nan=0.0) @ vf
            # weights and result are rounded to bf16 (2^-9 each) of values up to max|O|
            assert (out[0, x, r0:r1].float() - ref).abs().max().item() <= 1e-2 * ref.abs().max().clamp(min=1e-3).item()


# rows beyond whole rounds of workgroups, four, three and two pieces each; a head's last tile ragged; 1 row beyond a round
@pytest.mark.parametrize("heads,tokens,each", [(9, 128 * 58 - 31, 4), (19, 128 * 27, 4), (12, 128 * 110 + 5, 3), (5, 128 * 161, 3),
                                               (7, 128 * 128, 2)])
@pytest.mark.parametrize("flags", [0, 2])
def test_rows_beyond_whole_rounds(heads, tokens, each, flags):
    """Step 0, whose last rows on every XCD are cut, and a step that skips, on sampled rows and on rows cut and not cut of every
    XCD against the oracle; then the counters of both steps against the masks."""
    from paper_2511_11062_amd import lite_attn as la
    path = path_of(heads, tokens, flags)
    cut, share = path.pieces >> 4, -(-path.rows // 8)
    assert path.pieces & 15 == each and cut == -(-(path.rows % 512) // 8)
    ends = sorted({min(path.rows - 1, r) for x in range(0, 8, 3)
                   for r in (x * share + share - cut - 1, x * share + share - cut, x * share + share - 1)})
    wl = layer(heads, tokens, 0)
    reps = parity.run_sequence_check(wl, steps=2, thresholds=[-1.5, -0.8], diagonal_first=bool(flags), sample_rows=8, seed=flags,
                                     extra_rows=ends)
    assert reps[-1]["skipped_out"] > 0.02
    seq = inputs.DriftSequence(wl, "cuda:0")
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=2, flags=flags)
    try:
        la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
        outs, skipped = [], 0
        for t in range(2):
            q, k, v = (x.contiguous() for x in next(seq))
            for again in range(2 if t == 0 else 1):           # the same step 0 twice: the same bits, whatever piece came last
                out = torch.full_like(q, float("nan"))
                la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, -1.0, t)
                outs.append(out)
            st = la.lite_attn_skip_stats(h, t)
            mask = parity.unpack_mask(la.lite_attn_mask_export(h).reshape(path.rows, path.W), path.Tk)
            assert torch.isfinite(out).all()
            assert st.tiles_skipped_in == skipped and st.tiles_newly_marked == int(mask.sum()) - skipped
            skipped = int(mask.sum())
        assert skipped > 0 and torch.equal(outs[0], outs[1])
    finally:
        la.lite_attn_free_mask(h)
    # the allocation-free entry point learns from the mask itself that it is empty, and cuts the same rows
    desc = la.make_desc(1, heads, tokens, max_steps=1, flags=flags)
    mask = torch.zeros(la.static_mask_words(desc), dtype=torch.int64, device="cuda")
    seq = inputs.DriftSequence(wl, "cuda:0")
    for t in range(2):
        q, k, v = (x.contiguous() for x in next(seq))
        out = torch.full_like(q, float("nan"))
        la.lite_attn_fwd_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), desc, mask.data_ptr(), -1.0,
                                torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(out, outs[2 * t])


@pytest.mark.parametrize("heads,tokens,pieces", [(9, 128 * 15, 256), (10, 128 * 29 + 1, 512), (1, 128 * 129 + 7, 256)])
def test_pieces_on_a_busy_chip(heads, tokens, pieces):
    """Two handles on two streams, each with workgroups enough for the whole chip: many start when others of their call have ended
    and marked their rows.  Same outputs, masks and counters, bit for bit, as with the chip to itself."""
    from paper_2511_11062_amd import lite_attn as la
    path = path_of(heads, tokens)
    assert path.pieces == pieces
    wl = layer(heads, tokens, 0)
    seq = inputs.DriftSequence(wl, "cuda:0")
    data = [tuple(x.contiguous() for x in next(seq)) for _ in range(3)]
    thresholds = [-2.0, -1.2, -0.6]

    def trajectories(streams, rounds):
        handles = [la.lite_attn_init_mask(1, heads, tokens, max_steps=3) for _ in streams]
        outs = [[torch.full_like(data[0][0], float("nan")) for _ in data] for _ in streams]
        torch.cuda.synchronize()
        try:
            for h, s in zip(handles, streams):
                la.lite_attn_set_stream(h, s.cuda_stream)
            for _ in range(rounds):
                for t, (q, k, v) in enumerate(data):
                    for h, o in zip(handles, outs):
                        la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o[t].data_ptr(), h, thresholds[t], t)
            torch.cuda.synchronize()
            return [(o, la.lite_attn_mask_export(h), [la.lite_attn_skip_stats(h, t).tiles_newly_marked for t in range(3)])
                    for h, o in zip(handles, outs)]
        finally:
            for h in handles:
                la.lite_attn_free_mask(h)

    alone = trajectories([torch.cuda.Stream()], 1)[0]
    assert min(alone[2]) > 0
    for out, mask, newly in trajectories([torch.cuda.Stream(), torch.cuda.Stream()], 6):
        assert all(torch.equal(a, b) for a, b in zip(out, alone[0]))
        assert np.array_equal(mask, alone[1]) and newly == alone[2]


def test_import_goes_on_as_the_trajectory_would():
    """A step after an import of the mask gives what it gives in the trajectory that left the mask."""
    from paper_2511_11062_amd import lite_attn as la
    heads, tokens = 9, 128 * 15
    seq = inputs.DriftSequence(layer(heads, tokens, 0), "cuda:0")
    data = [tuple(x.contiguous() for x in next(seq)) for _ in range(3)]
    h, g = (la.lite_attn_init_mask(1, heads, tokens, max_steps=3) for _ in range(2))
    try:
        for x in (h, g):
            la.lite_attn_set_stream(x, torch.cuda.current_stream().cuda_stream)
        outs = [torch.full_like(data[0][0], float("nan")) for _ in data]
        for t, (q, k, v) in enumerate(data):
            mask = la.lite_attn_mask_export(h)
            la.lite_attn_skipruns_export(h, heads * 15)        # (leaves what the next call needs alone)
            la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), outs[t].data_ptr(), h, [-2.0, -1.2, -0.6][t], t)
            if t == 0:
                continue
            out = torch.full_like(q, float("nan"))
            la.lite_attn_mask_import(g, mask, t)
            la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), g, [-2.0, -1.2, -0.6][t], t)
            assert torch.equal(out, outs[t])
            assert np.array_equal(la.lite_attn_mask_export(g), la.lite_attn_mask_export(h))
    finally:
        for x in (h, g):
            la.lite_attn_free_mask(x)


# whole rows and two to seven equal segments, in pairs and in single groups; more segments than run side by side (4 x 87: 1392);
# protected rows of the literal skip
@pytest.mark.parametrize("heads,tokens,flags,text,nseg", [
    (9, 128 * 15 - 3, 0, 0, 1), (10, 128 * 29, 2, 0, 1), (6, 128 * 20, 2, 0, 2), (4, 128 * 86, 0, 0, 2), (5, 128 * 16 - 9, 0, 0, 3),
    (3, 128 * 27, 0, 0, 3), (3, 128 * 35, 2, 50, 4), (2, 128 * 64 - 1, 0, 0, 4), (4, 128 * 87, 0, 0, 4), (4, 128 * 25 - 70, 0, 0, 5),
    (4, 128 * 70, 0, 0, 5), (1, 128 * 129 + 7, 0, 0, 7), (1, 128 * 180, 2, 0, 7), (5, 128 * 31 - 55, 3, 100, 1)])
def test_empty_mask_however_the_caller_came_by_it(heads, tokens, flags, text, nseg):
    """The first call of a handle, later calls on a mask that is still empty (known to be, or not), a call on an imported empty
    mask and the allocation-free call: the same bits out of all of them, and the same mask behind."""
    from paper_2511_11062_amd import lite_attn as la
    wl = layer(heads, tokens, text)
    path = path_of(heads, tokens, flags, wl.protect)
    assert path.pieces > 0 and path.nseg == nseg
    q, k, v = (x.contiguous() for x in next(inputs.DriftSequence(wl, "cuda:0")))
    stream = torch.cuda.current_stream().cuda_stream
    fields = {"max_steps": 2, "flags": flags, "protect": wl.protect}
    results = {}

    def call(h, threshold, step):
        out = torch.full_like(q, float("nan"))
        la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, threshold, step)
        return out

    for way, before in (("first", None), ("known empty", -float("inf")), ("nothing marked", -1e30), ("import", 0)):
        h = la.lite_attn_init_mask(1, heads, tokens, **fields)
        try:
            la.lite_attn_set_stream(h, stream)
            if way == "import":
                la.lite_attn_mask_import(h, np.zeros(la.lite_attn_mask_words(h), np.uint64), 1)
            elif before is not None:
                call(h, before, 0)
            step = 0 if before is None else 1
            out = call(h, -1.0, step)
            st = la.lite_attn_skip_stats(h, step)
            results[way] = out, la.lite_attn_mask_export(h)
            marked = int(parity.unpack_mask(results[way][1].reshape(path.rows, path.W), path.Tk).sum())
            assert st.tiles_skipped_in == 0 and st.tiles_newly_marked == marked > 0, way
        finally:
            la.lite_attn_free_mask(h)
    desc = la.make_desc(1, heads, tokens, **fields)
    mask = torch.zeros(la.static_mask_words(desc), dtype=torch.int64, device="cuda")
    out = torch.full_like(q, float("nan"))
    la.lite_attn_fwd_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), desc, mask.data_ptr(), -1.0, stream)
    torch.cuda.synchronize()
    results["static"] = out, mask.cpu().numpy().view(np.uint64)
    first = results.pop("first")
    assert torch.isfinite(first[0]).all()
    for way, (o, m) in results.items():
        assert np.array_equal(m, first[1]), way
        assert torch.equal(o, first[0]), (way, int((o != first[0]).sum()))


@pytest.mark.parametrize("heads,tokens,flags", [(9, 128 * 58 - 31, 0), (12, 128 * 110 + 5, 2), (7, 128 * 128, 0)])
def test_later_steps_on_a_mask_known_to_be_empty(heads, tokens, flags):
    """More rows than run side by side, two dense steps, then steps that mark: the third finds an empty mask without a schedule,
    cuts the last rows and judges them.  Its bits are those of a new handle's first call; the fourth's those of a call on the
    imported mask; masks and counters of every step."""
    from paper_2511_11062_amd import lite_attn as la
    path = path_of(heads, tokens, flags)
    assert path.rows > 512 and path.pieces & 15 > 1
    seq = inputs.DriftSequence(layer(heads, tokens, 0), "cuda:0")
    data = [tuple(x.contiguous() for x in next(seq)) for _ in range(2)]
    data = [data[0], data[1], data[0], data[1]]
    thresholds = [-float("inf"), -float("inf"), -1.0, -0.8]
    handles = [la.lite_attn_init_mask(1, heads, tokens, max_steps=4, flags=flags) for _ in range(3)]
    outs, masks = [], []

    def call(h, t, step):
        out = torch.full_like(data[t][0], float("nan"))
        la.lite_attn_fwd(*(x.data_ptr() for x in data[t]), out.data_ptr(), h, thresholds[t], step)
        return out

    try:
        for h in handles:
            la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
        for t in range(4):
            outs.append(call(handles[0], t, t))
            st = la.lite_attn_skip_stats(handles[0], t)
            masks.append(la.lite_attn_mask_export(handles[0]))
            marked = [int(parity.unpack_mask(m.reshape(path.rows, path.W), path.Tk).sum()) for m in masks]
            before = marked[-2] if t else 0
            assert st.tiles_skipped_in == before and st.tiles_newly_marked == marked[-1] - before
            assert torch.isfinite(outs[-1]).all()
        assert marked[1] == 0 < marked[2] < marked[3]
        assert torch.equal(call(handles[1], 2, 0), outs[2])
        assert np.array_equal(la.lite_attn_mask_export(handles[1]), masks[2])
        la.lite_attn_mask_import(handles[2], masks[2], 3)
        assert torch.equal(call(handles[2], 3, 3), outs[3])
        assert np.array_equal(la.lite_attn_mask_export(handles[2]), masks[3])
    finally:
        for h in handles:
            la.lite_attn_free_mask(h)


# more equal pieces than four, and more of them than run side by side: pairs (three of each row), single groups (three, four, five)
@pytest.mark.parametrize("heads,tokens,equal", [(1, 128 * 129 + 7, 3), (5, 128 * 60 - 1, 3), (4, 128 * 87, 4), (1, 128 * 202 - 64, 5)])
def test_rows_cut_alike_under_a_mask(heads, tokens, equal):
    """15 % of every row's tiles skipped, which leaves no room for pieces of the rows' own: outputs against block-masked softmax
    in fp32, marks against the predicate, whose running maximum goes through all pieces; twice with the same bits."""
    from paper_2511_11062_amd import lite_attn as la
    path = path_of(heads, tokens)
    tiles, thr = path.Tk, -1.0
    assert path.pieces > 0 and heads * tiles * equal > path.pieces
    rng = np.random.default_rng(tokens)
    skip = rng.random((heads, tiles, tiles)) < 0.15
    g = torch.Generator(device="cuda").manual_seed(tokens)
    q, k, v = (torch.randn(1, heads, tokens, 128, device="cuda", generator=g) for _ in range(3))
    # tiles of keys that lie far off for all queries, so that some fire
    far = torch.from_numpy(rng.random(tiles) < 0.3).cuda().repeat_interleave(128)[:tokens]
    q[..., 0], k[..., 0] = 4.0, torch.where(far, -12.0, 2.0)
    q, k, v = (x.to(torch.bfloat16).contiguous() for x in (q, k, v))
    packed = parity.pack_mask(skip.astype(np.uint8))
    h = la.lite_attn_init_mask(1, heads, tokens, max_steps=2)
    la.lite_attn_set_stream(h, torch.cuda.current_stream().cuda_stream)
    outs, masks = [], []
    try:
        for _ in range(2):
            out = torch.full_like(q, float("nan"))
            la.lite_attn_mask_import(h, packed, 1)
            la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), h, thr, 1)
            masks.append(la.lite_attn_mask_export(h))
            outs.append(out)
    finally:
        la.lite_attn_free_mask(h)
    assert torch.equal(outs[0], outs[1]) and np.array_equal(masks[0], masks[1])
    marked = torch.from_numpy(parity.unpack_mask(masks[0].reshape(heads, tiles, path.W), tiles)).cuda().bool()
    dead = torch.from_numpy(skip).cuda()
    assert bool((marked | ~dead).all()) and int((marked & ~dead).sum()) > 50 * heads
    for x in range(heads):
        kf, vf = k[0, x].float().t().contiguous(), v[0, x].float()
        for i0 in range(0, tiles, 32):
            n, r0, r1 = min(32, tiles - i0), 128 * i0, min(tokens, 128 * (i0 + 32))
            s = torch.full((128 * n, 128 * tiles), -float("inf"), device="cuda")
            s[:r1 - r0, :tokens] = (q[0, x, r0:r1].float() @ kf) * 128 ** -0.5
            s4 = s.view(n, 128, tiles, 128).masked_fill_(dead[x, i0:i0 + n][:, None, :, None], -float("inf"))
            mloc = s4.amax(dim=3)
            gap = mloc - mloc.cummax(dim=2).values                               # NaN where nothing has been visited yet
            gap[(torch.arange(128 * n, device="cuda") + r0 >= tokens).view(n, 128)] = -float("inf")
            worst = gap.amax(dim=1)
            here, gone = marked[x, i0:i0 + n], dead[x, i0:i0 + n]
            clear = ~gone & ((worst - thr).abs() > parity.G_BAND)
            assert torch.equal(here[clear], worst[clear] <= thr)
            ref = torch.softmax(s[:r1 - r0], dim=1)[:, :tokens] @ vf
            # weights and result are rounded to bf16 (2^-9 each) of values up to max|O|
            assert (outs[0][0, x, r0:r1].float() - ref).abs().max().item() <= 1e-2 * ref.abs().max().item()
