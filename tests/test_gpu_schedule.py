"""Row schedules: every row exactly once, and no XCD with more than its share of the work, however uneven the heads are.
Workgroups go to XCDs by id, so the busiest XCD's work is the step's time."""
import ctypes

import numpy as np
import pytest
import torch

import parity

pytestmark = pytest.mark.gpu
ROW_OVERHEAD = 2        # what a row costs besides its tiles, in tile times


def schedule_of_short_rows(skip):
    """The table that schedule_rows_kernel makes of a mask [heads, tiles, tiles]: a list of row ids per XCD."""
    from paper_2511_11062_amd import lite_attn as la
    heads, tiles = skip.shape[:2]
    path = parity.path_of(1, heads, 128 * tiles)
    rows = heads * tiles
    assert path.nseg == 1 and rows > 512, "not a shape with a one-launch schedule"
    bits = torch.from_numpy(parity.pack_mask(skip.astype(np.uint8)).reshape(rows, -1).view(np.int64)).cuda()
    slots = torch.full((8, path.per_xcd), -1, dtype=torch.int32, device="cuda")
    used = torch.full((8,), -1, dtype=torch.int32, device="cuda")
    launch = la._lib._ZN2la20launch_schedule_rowsEPKmiiiiPjS2_P12ihipStream_t
    launch.restype = ctypes.c_int
    launch.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 4 + [ctypes.c_void_p] * 3
    assert launch(bits.data_ptr(), rows, tiles, bits.shape[1], path.per_xcd, slots.data_ptr(), used.data_ptr(),
                  torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    table, used = slots.cpu().numpy(), used.cpu().numpy()
    assert (used >= 0).all() and (used <= path.per_xcd).all()
    return [table[x, :used[x]] for x in range(8)]


def halves(heads, a, b):
    return np.where(np.arange(heads) < heads // 2, a, b)


# live share of each head: alike; the first half of the heads longer than the second (two halves of a batch, say); the
# same interleaved; one head, or an eighth of them, with nearly all of the work; heads that skip everything
@pytest.mark.parametrize("heads,tiles,live", [
    (24, 37, np.full(24, 0.4)), (9, 57, np.full(9, 0.5)), (40, 61, halves(40, 0.9, 0.3)), (40, 61, halves(40, 0.7, 0.2)),
    (40, 61, halves(40, 0.9, 0.15)), (24, 37, halves(24, 0.15, 0.9)), (40, 61, np.where(np.arange(40) % 2, 0.2, 0.7)),
    (8, 128, np.where(np.arange(8) == 0, 0.95, 0.05)), (8, 192, np.where(np.arange(8) == 5, 1.0, 0.0)),
    (12, 110, np.where(np.arange(12) < 2, 1.0, 0.02)), (40, 128, np.where(np.arange(40) < 5, 1.0, 0.01)),
    (170, 192, halves(170, 0.0, 1.0)), (520, 2, np.where(np.arange(520) < 65, 1.0, 0.0)), (513, 1, np.full(513, 1.0)),
    (27, 19, np.zeros(27)), (32768, 1, halves(32768, 1.0, 0.0)), (16, 64, np.linspace(0.0, 1.0, 16))])
def test_equal_work_on_every_xcd(heads, tiles, live):
    rng = np.random.default_rng(heads * tiles)
    skip = rng.random((heads, tiles, tiles)) >= live[:, None, None]
    xcds = schedule_of_short_rows(skip)
    assert np.array_equal(np.sort(np.concatenate(xcds)), np.arange(heads * tiles))
    count = (~skip).sum(axis=2).reshape(-1)
    work = np.array([(count[rows] + ROW_OVERHEAD).sum() for rows in xcds])
    # a share may end inside a row: one row too many at its end, one too few at its start
    assert work.max() <= work.mean() + 2 * (tiles + ROW_OVERHEAD), work / work.mean()
    for rows in xcds:                                       # long rows first, to within a class (a 32nd of a row)
        assert (np.diff(count[rows]) <= tiles // 32 + 1).all()
