"""What the launch code takes for granted about every layer whose rows may be shared by several workgroups, over all of them:
compiled from the library's own host code, without a GPU."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <algorithm>
#include "lite_attn_kernels.h"
using namespace la;
struct Most { long layers, scratch, with_lists, equal, parts_end, tiles; };
// Largest values over the layers of first..last rows that cut rows, heads and tiles in every way.
extern "C" Most most(int first, int last, int flags) {
  Most m = {};
  for (int Tk = 1; Tk <= (last > kFewRows ? kShortTiles : last); ++Tk)
    for (int heads = std::max(1, (first + Tk - 1) / Tk); heads * Tk <= last; ++heads) {
      const lite_attn_desc_t d = {1, heads, 128 * Tk, 128, 128, 128, (int64_t)heads * Tk * 16384, (int64_t)Tk * 16384, 128,
                                  0, 1, flags, 1};
      const Geometry g = geometry(d);
      if (g.pieces == 0 && g.nseg <= 1) continue;
      const long total = (long)scratch_layout(g).total;
      ++m.layers;
      m.scratch = std::max(m.scratch, total);
      m.with_lists = std::max(m.with_lists, (long)list_layout(g).total + total);
      if (g.pieces == 0) continue;
      m.equal = std::max(m.equal, (long)equal_pieces(g));
      m.tiles = std::max(m.tiles, (long)g.Tk);
      // the row maxima of the last row that has some, behind the partial results, with either kind of cut
      const long rows = g.rows > kFewRows ? 8l * cut_rows(g) : (long)g.rows;
      for (int n : {1, g.rows > kFewRows ? 1 : equal_pieces(g), g.rows > kFewRows ? 1 : g.nseg}) {
        const ScratchLayout s = scratch_layout(g, n);
        m.parts_end = std::max(m.parts_end, (long)s.seg_mloc + 4 * rows * g.Tk * 128 - total);
        const long parts = n > 1 ? g.rows * n : g.rows > kFewRows ? rows * cut_pieces(g)
                                                                  : std::max<long>(g.pieces, g.rows * equal_pieces(g));
        m.parts_end = std::max(m.parts_end, std::max(4 * parts * 128 * 128 - (long)s.seg_stat,
                                                     (long)s.seg_stat + 4 * parts * 2 * 128 - (long)s.seg_mloc));
      }
    }
  return m;
}
extern "C" long limit() { return (long)kMaxSegmentBytes; }
extern "C" long array() { return (long)LITE_ATTN_STATIC_SCRATCH_BYTES; }
"""


class Most(ctypes.Structure):
    _fields_ = [(n, ctypes.c_long) for n in ("layers", "scratch", "with_lists", "equal", "parts_end", "tiles")]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("scratch")
    (d / "most.cpp").write_text(SRC)
    csrc = os.path.join(ROOT, "paper_2511_11062_amd", "csrc")
    out = str(d / "libmost.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "tests", "hip_stub"),
                    "-I" + os.path.join(ROOT, "include"), "-I" + csrc, str(d / "most.cpp"),
                    os.path.join(csrc, "lite_attn_host.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.most.restype, lib.limit.restype, lib.array.restype = Most, ctypes.c_long, ctypes.c_long
    return lib


@pytest.mark.parametrize("flags", [0, 1, 2, 3])
@pytest.mark.parametrize("first,last", [(1, 512), (513, 32768)])
def test_partial_results_fit_for_every_layer(lib, first, last, flags):
    m = lib.most(first, last, flags)
    assert (m.layers > 0) == (last == 512 and flags != 1 or flags in (0, 2))   # the literal skip cuts protected rows alone
    assert m.scratch <= lib.limit()                  # what the header promises, and
    assert m.with_lists <= lib.array()               # the allocation-free entry point takes every layer that a handle cuts
    assert m.equal <= 15                             # four bits of the word that the kernel keeps them in
    assert m.parts_end <= 0                          # nothing runs into what lies behind it
    assert m.tiles < 1 << 15                         # tiles of a row in 16 bits of a Skip-List entry
