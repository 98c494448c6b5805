"""GPU-vs-oracle comparison of the skip-aware attention path (used by the gpu tests and the smoke check).

Protocol: the oracle runs its own mask trajectory (its inputs never come from the HIP path).  Before every
step the oracle's entry mask is imported into the HIP handle for the compared rows ("teacher forcing"), so
that one borderline tile cannot change the inputs of later steps; then both run the step on the same
bf16 bytes and are compared:
  * output: max|dO| <= 1e-2 * max|O| and mean|dO| <= 1e-3;
  * exit mask: bit-exact, except tiles whose oracle predicate value lies within 1e-3 of the threshold.
Rows (b,h,i) are independent, so large shapes are compared on a sample of rows.
"""
import ctypes

import numpy as np
import torch

from paper_2511_11062_amd import inputs
from oracle.lite_attn_oracle import oracle_step

MAX_REL = 1e-2     # max|dO| <= MAX_REL * max|O|
MEAN_ABS = 1e-3    # mean|dO| <= MEAN_ABS
G_BAND = 1e-3      # |g - thr| <= G_BAND excuses a mask bit


class Path(ctypes.Structure):
    """la::Geometry (csrc/lite_attn_kernels.h): which way through the library a shape takes.  nseg 0: Skip-Lists, row
    ranking and V^T; 1: whole rows found from the mask; more: rows cut into segments.  pair: workgroups of two groups."""
    _fields_ = [("Tq", ctypes.c_int), ("Tk", ctypes.c_int), ("W", ctypes.c_int), ("run_stride", ctypes.c_int),
                ("BH", ctypes.c_int), ("rows", ctypes.c_int64), ("chunks", ctypes.c_int), ("pair", ctypes.c_int),
                ("nseg", ctypes.c_int), ("per_xcd", ctypes.c_int)]


def path_of(batch, heads, seqlen, flags=0) -> Path:
    """What the library itself decides for a layer, so that a test can say which kernels it is about."""
    from paper_2511_11062_amd import lite_attn as la
    f = la._lib._ZN2la8geometryERK16lite_attn_desc_t
    f.restype, f.argtypes = Path, [ctypes.POINTER(la.Desc)]
    p = f(ctypes.byref(la.make_desc(batch, heads, seqlen, flags=flags)))
    assert (p.Tk, p.BH, p.rows) == (-(-seqlen // 128), batch * heads, batch * heads * -(-seqlen // 128))
    return p


def pack_mask(mask_bytes: np.ndarray) -> np.ndarray:
    """uint8 [..., Tk] (nonzero = skipped) -> uint64 [..., ceil(Tk/64)], bit j%64 of word j/64."""
    tk = mask_bytes.shape[-1]
    w = -(-tk // 64)
    padded = np.zeros(mask_bytes.shape[:-1] + (w * 64,), dtype=np.uint8)
    padded[..., :tk] = mask_bytes != 0
    b = np.packbits(padded, axis=-1, bitorder="little")
    return np.ascontiguousarray(b).view(np.uint64)


def unpack_mask(bits: np.ndarray, tk: int) -> np.ndarray:
    """inverse of pack_mask: uint64 [..., W] -> uint8 [..., tk]"""
    by = np.ascontiguousarray(bits).view(np.uint8)
    return np.unpackbits(by, axis=-1, bitorder="little")[..., :tk]


def compare_output(o_gpu: np.ndarray, o_ref: np.ndarray):
    d = np.abs(o_gpu.astype(np.float64) - o_ref.astype(np.float64))
    return float(d.max()), float(d.mean()), float(np.abs(o_ref).max())


def check_step(o_gpu, o_ref, m_gpu, m_ref, g_ref, thr, o_keep=None):
    """Raises AssertionError on a parity violation; returns a small report dict.  o_keep: optional boolean selector
    of the output rows to compare (immediate mode leaves out Q tiles that have a mask bit excused by the band: there
    the two sides may legitimately have dropped different tiles from the output)."""
    if o_keep is not None:
        o_gpu, o_ref = o_gpu[o_keep], o_ref[o_keep]
    mx, mean, omax = compare_output(o_gpu, o_ref)
    assert np.isfinite(o_gpu).all(), "non-finite output"
    assert mx <= MAX_REL * omax, "max|dO| = %.3e > %.1e * max|O| (%.3e)" % (mx, MAX_REL, omax)
    assert mean <= MEAN_ABS, "mean|dO| = %.3e > %.1e" % (mean, MEAN_ABS)
    diff = (m_gpu != 0) != (m_ref != 0)
    with np.errstate(invalid="ignore"):
        excused = np.abs(g_ref - thr) <= G_BAND      # NaN (tile not evaluated) is never excused
    bad = diff & ~excused
    assert not bad.any(), "%d mask bits differ outside the +-%.0e band (first at %s)" % (
        int(bad.sum()), G_BAND, tuple(np.argwhere(bad)[0]))
    return {"max_dO": mx, "mean_dO": mean, "max_O": omax, "mask_excused": int((diff & excused).sum()),
            "skipped_out": float((m_ref != 0).mean())}


def run_sequence_check(workload, steps=None, threshold=-2.0, thresholds=None, sample_rows=None, gen_device=None,
                       verbose=False, seed=0, layout="bhnd", diagonal_first=False, immediate=False,
                       free_running=False, extra_rows=(), say=print):
    """Runs `steps` denoising steps of a named workload on cuda:0 through the C ABI and checks every step.

    sample_rows: None = all rows; an int = that many seeded random rows plus first/last (and protected) rows, plus
    `extra_rows` (flattened row ids (b*H+h)*Tq+i).  say: where the verbose per-step lines go.
    immediate: both sides drop a fired tile in the call that marks it (Algorithm 2 literally).
    free_running: no teacher forcing -- the HIP path keeps its own mask trajectory.  A compared Q tile whose two entry
    masks still agree is checked as usual (so the first disagreement of a row has to lie inside the band); rows whose
    trajectories have parted are only counted ("diverged_rows", "diverged_bits" in the report).
    Returns the list of per-step reports."""
    from paper_2511_11062_amd import lite_attn as la
    wl = inputs.WORKLOADS[workload] if isinstance(workload, str) else workload
    steps = steps or wl.steps
    dev = torch.device("cuda:0")
    B, H, N, d = wl.batch, wl.heads, wl.seqlen, wl.head_dim
    Tq = Tk = -(-N // 128)
    W = -(-Tk // 64)
    if sample_rows is None:
        rows = np.arange(B * H * Tq)
    else:
        rng = np.random.default_rng(seed)
        base = {0, Tq - 1, B * H * Tq - 1, (B * H - 1) * Tq}
        if wl.text_tokens:
            base |= {wl.video_tokens // 128, wl.video_tokens // 128 - 1, Tq + wl.video_tokens // 128}
        base = {r for r in base if 0 <= r < B * H * Tq}          # (a single head has no second head's text rows)
        rows = np.array(sorted(base | set(int(r) for r in extra_rows) |
                               set(rng.choice(B * H * Tq, size=sample_rows, replace=False).tolist())))
    assert rows.min() >= 0 and rows.max() < B * H * Tq
    heads = sorted({int(r // Tq) for r in rows})            # flattened (b*H+h)
    head_pos = {bh: n for n, bh in enumerate(heads)}
    sub_rows = [head_pos[int(r // Tq)] * Tq + int(r % Tq) for r in rows]

    seq = inputs.DriftSequence(wl, gen_device or ("cpu" if B * H * N <= 1 << 16 else dev))
    # "bnhd": memory order [B,N,H,d]; "padded": [B,H,N,d+8] with 8 unused elements after every token row, and a gap
    # of 64 elements after every head
    pad_n, pad_h = d + 8, N * (d + 8) + 64
    strides = {"bhnd": None, "bnhd": (N * H * d, d, H * d), "padded": (H * pad_h, pad_h, pad_n)}[layout]
    handle = la.lite_attn_init_mask(B, H, N, protect=wl.protect, max_steps=max(steps, 1), strides=strides,
                                    flags=(la.LITE_ATTN_ORDER_DIAGONAL_FIRST if diagonal_first else 0) |
                                    (la.LITE_ATTN_PV_SKIP_IMMEDIATE if immediate else 0))
    visit = None
    if diagonal_first:
        from oracle.lite_attn_oracle import diagonal_first as diag
        visit = diag(Tq, Tk)
    la.lite_attn_set_stream(handle, torch.cuda.current_stream().cuda_stream)
    m_ref = np.zeros((1, len(heads), Tq, Tk), dtype=np.uint8)      # oracle mask of the compared heads
    m_gpu = np.zeros((len(rows), Tk), dtype=np.uint8)              # HIP mask of the compared rows after the last step
    reports = []
    try:
        for t in range(steps):
            thr = thresholds[t] if thresholds is not None else threshold
            q, k, v = (x.to(dev).contiguous() for x in next(seq))
            if layout == "bnhd":
                mem = [x.permute(0, 2, 1, 3).contiguous() for x in (q, k, v)]
                out_mem = torch.empty_like(mem[0])
                out = out_mem.permute(0, 2, 1, 3)
            elif layout == "padded":
                def padded(x=None):
                    buf = torch.full((B * H * pad_h,), float("nan"), dtype=torch.bfloat16, device=dev)
                    view = torch.as_strided(buf, (B, H, N, d), (H * pad_h, pad_h, pad_n, 1))
                    if x is not None:
                        view.copy_(x)
                    view.whole_buffer = buf
                    return view
                mem = [padded(x) for x in (q, k, v)]                   # the gaps hold NaN: nothing may read them
                out_mem = out = padded()
            else:
                mem = [q, k, v]
                out_mem = out = torch.empty_like(q)
            qs, ks, vs = (inputs.bf16_bits(x.reshape(B * H, N, d)[heads].unsqueeze(0)) for x in (q, k, v))
            # teacher forcing: compared rows of the HIP mask := oracle's entry mask
            if t > 0 and not free_running:
                bits = la.lite_attn_mask_export(handle).reshape(B * H * Tq, W)
                bits[rows] = pack_mask(m_ref.reshape(-1, Tk)[sub_rows])
                la.lite_attn_mask_import(handle, bits, t)
            la.lite_attn_fwd(mem[0].data_ptr(), mem[1].data_ptr(), mem[2].data_ptr(), out_mem.data_ptr(), handle,
                             thr, t)
            torch.cuda.synchronize()
            same = (m_gpu != 0) == (m_ref.reshape(-1, Tk)[sub_rows] != 0)       # entry masks, per compared row
            row_ok = same.all(axis=1) if free_running else np.ones(len(rows), dtype=bool)
            o_ref, m_new, g = oracle_step(qs, ks, vs, m_ref, thr, protect=wl.protect, rows=sub_rows, visit=visit,
                                          immediate=immediate)
            o_gpu = out.reshape(B * H, N, d)[heads].float().cpu().numpy()
            if layout == "padded":                                     # nothing was written into the gaps of `out`
                untouched = torch.isnan(out.whole_buffer.float())
                torch.as_strided(untouched, (B, H, N, d), (H * pad_h, pad_h, pad_n, 1)).fill_(True)
                assert bool(untouched.all()), "the kernel wrote outside the rows of `out`"
            m_gpu = unpack_mask(la.lite_attn_mask_export(handle).reshape(B * H * Tq, W), Tk)[rows]
            sel_o = np.zeros((len(heads), N), dtype=bool)
            for r in sub_rows:
                sel_o[r // Tq, (r % Tq) * 128:min(N, (r % Tq + 1) * 128)] = True
            g_rows = g.reshape(-1, Tk)[sub_rows]
            o_keep = None
            if immediate or free_running:
                with np.errstate(invalid="ignore"):
                    near = (np.abs(g_rows - thr) <= G_BAND).any(axis=1)        # per compared Q tile, in sub_rows order
                if not immediate:
                    near[:] = False
                keep_tile = {r: bool(ok and not n) for r, n, ok in zip(sub_rows, near, row_ok)}
                tile_of_token = np.zeros((len(heads), N), dtype=np.int64)
                tile_of_token[:] = np.arange(N) // 128
                tile_of_token += (np.arange(len(heads)) * Tq)[:, None]
                o_keep = np.array([keep_tile[int(x)] for x in tile_of_token[sel_o]])
            m_exit = m_new.reshape(-1, Tk)[sub_rows]
            rep = check_step(o_gpu[sel_o], o_ref[0][sel_o], m_gpu[row_ok], m_exit[row_ok], g_rows[row_ok], thr, o_keep)
            rep.update(diverged_rows=int((~row_ok).sum()), diverged_bits=int(((m_gpu != 0) != (m_exit != 0)).sum()))
            st = la.lite_attn_skip_stats(handle, t)
            rep.update(step=t, threshold=thr, gpu_skipped_in=st.tiles_skipped_in / st.tiles_total,
                       gpu_newly=st.tiles_newly_marked / st.tiles_total, rows=len(rows))
            if verbose:
                say("step %d thr %.2f, %d rows: max|dO| %.2e (max|O| %.2f) mean|dO| %.2e, skipped-out %.3f, excused %d" % (
                    t, thr, len(rows), rep["max_dO"], rep["max_O"], rep["mean_dO"], rep["skipped_out"],
                    rep["mask_excused"]))
            reports.append(rep)
            m_ref = m_new
    finally:
        la.lite_attn_free_mask(handle)
    return reports
