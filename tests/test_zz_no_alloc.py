"""The allocation-free entry point against the handle-based one (needs an MI355X).  Collected last on purpose."""
import numpy as np
import pytest
import torch

import parity
from paper_2511_11062_amd import inputs
from paper_2511_11062_amd import lite_attn as la

pytestmark = pytest.mark.gpu


def _layer(name, heads, grid, seed, text=0):
    wl = inputs.Workload(name, 1, heads, grid, text_tokens=text, steps=2, seed=seed)
    seq = inputs.DriftSequence(wl, "cpu")
    return wl, [tuple(x.cuda().contiguous() for x in next(seq)) for _ in range(2)]


def test_static_entry_point_matches_the_handle_path():
    """lite_attn_fwd_static on layers in a row, each smaller than the one before (so the static array still holds
    that one's Skip-List, row schedule, V^T or partial results beyond what the next overwrites), two timesteps each with the
    caller-owned Skip-Mask carried from the first to the second: outputs and masks must equal what lite_attn_fwd
    gives with a handle -- the same kernels on the same inputs, so bit for bit, which is inside every tolerance."""
    stream = torch.cuda.current_stream().cuda_stream
    thr = [-3.0, -2.0]
    # Skip-Lists and V^T, rows scheduled from the mask, segments: N = 24699, 5100, 1528, 300
    layers = [_layer("na_lists", 3, (5, 60, 82), 54, text=99), _layer("na_schedule", 16, (3, 40, 42), 55, text=60),
              _layer("na_big", 3, (2, 24, 31), 51, text=40), _layer("na_small", 2, (1, 12, 25), 52)]
    assert [parity.path_of(1, wl.heads, wl.seqlen).nseg > 0 for wl, _ in layers] == [False, True, True, True]
    for wl, data in layers:
        H, N = wl.heads, wl.seqlen
        h = la.lite_attn_init_mask(1, H, N, protect=wl.protect, max_steps=2)
        la.lite_attn_set_stream(h, stream)
        ref = []
        try:
            for t, (q, k, v) in enumerate(data):
                o = torch.empty_like(q)
                la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), h, thr[t], t)
                torch.cuda.synchronize()
                ref.append((o, la.lite_attn_mask_export(h).copy()))
        finally:
            la.lite_attn_free_mask(h)
        desc = la.make_desc(1, H, N, protect=wl.protect, max_steps=1)
        mask = torch.zeros(la.static_mask_words(desc), dtype=torch.int64, device="cuda")     # the caller's Skip-Mask
        for t, (q, k, v) in enumerate(data):
            o = torch.full_like(q, float("nan"))
            la.lite_attn_fwd_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), desc, mask.data_ptr(),
                                    thr[t], stream)
            torch.cuda.synchronize()
            got_mask = mask.cpu().numpy().view(np.uint64)
            assert np.array_equal(got_mask, ref[t][1]), "%s step %d: Skip-Mask differs" % (wl.name, t)
            assert ref[t][1].any()
            d = (o.float() - ref[t][0].float()).abs()
            assert torch.isfinite(o).all()
            assert d.max().item() <= 1e-2 * ref[t][0].float().abs().max().item() and d.mean().item() <= 1e-3
            assert torch.equal(o, ref[t][0]), "%s step %d: output differs" % (wl.name, t)


def test_static_entry_point_takes_short_rows_whatever_the_size_of_v():
    """5120 rows of 128 tiles: V alone is larger than the static array, but such a call needs no copy of it.  A dense step
    and one that skips, bit for bit what a handle gives."""
    heads, n = 40, 128 * 128
    desc = la.make_desc(1, heads, n, max_steps=1)
    assert heads * n * 256 > 128 << 20
    g = torch.Generator(device="cuda").manual_seed(53)
    q, k, v = (torch.randn(1, heads, n, 128, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    q.mul_(3.0)                                                # peaked rows: some tiles fire at the threshold below
    stream = torch.cuda.current_stream().cuda_stream
    mask = torch.zeros(la.static_mask_words(desc), dtype=torch.int64, device="cuda")
    out, ref = torch.empty_like(q), torch.empty_like(q)
    h = la.lite_attn_init_mask(1, heads, n, max_steps=2)
    la.lite_attn_set_stream(h, stream)
    try:
        for t in range(2):
            la.lite_attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), ref.data_ptr(), h, -0.3, t)
            la.lite_attn_fwd_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.fill_(float("nan")).data_ptr(), desc,
                                    mask.data_ptr(), -0.3, stream)
            torch.cuda.synchronize()
            assert torch.equal(out, ref), "step %d" % t
            got = mask.cpu().numpy().view(np.uint64)
            assert np.array_equal(got, la.lite_attn_mask_export(h)) and got.any()
    finally:
        la.lite_attn_free_mask(h)


def test_static_entry_point_refuses_what_does_not_fit():
    wl = inputs.WORKLOADS["wan14b"]
    desc = la.make_desc(1, wl.heads, wl.seqlen)
    x = torch.zeros(64, dtype=torch.bfloat16, device="cuda")
    m = torch.zeros(8, dtype=torch.int64, device="cuda")
    with pytest.raises(la.LiteAttnError) as err:
        la.lite_attn_fwd_static(x.data_ptr(), x.data_ptr(), x.data_ptr(), x.data_ptr(), desc, m.data_ptr(), -1.0,
                                torch.cuda.current_stream().cuda_stream)
    assert err.value.code == -7
