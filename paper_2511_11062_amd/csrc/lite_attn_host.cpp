// Pure host logic of the C ABI (no HIP call, no device code): descriptor and call checks, tile geometry, layout of
// the per-call scratch.  Kept apart so that it also builds with a plain C++ compiler under the CPU sanitizers.
#include <algorithm>
#include <cmath>

#include "lite_attn_kernels.h"

namespace la {

int check_desc(const lite_attn_desc_t* d) {
  if (!d) return LITE_ATTN_EINVAL;
  if (d->batch < 1 || d->heads < 1 || d->seqlen < 1 || d->head_dim < 1 || d->tile_q < 1 || d->tile_k < 1)
    return LITE_ATTN_EINVAL;
  if (d->max_steps < 1) return LITE_ATTN_EINVAL;
  if ((d->flags & ~(LITE_ATTN_ORDER_DIAGONAL_FIRST | LITE_ATTN_PV_SKIP_IMMEDIATE)) != 0) return LITE_ATTN_EINVAL;
  if (d->protect_len < 0 || d->protect_start < 0 ||
      (d->protect_len > 0 && (int64_t)d->protect_start + d->protect_len > d->seqlen))
    return LITE_ATTN_EINVAL;
  // 16-byte vector accesses: every stride must be a multiple of 8 bf16 elements
  if (d->stride_n < d->head_dim || d->stride_b < 0 || d->stride_h < 0) return LITE_ATTN_EINVAL;
  if ((d->stride_n % 8) || (d->stride_b % 8) || (d->stride_h % 8)) return LITE_ATTN_EINVAL;
  if (d->batch > 1 && d->stride_b == 0) return LITE_ATTN_EINVAL;
  if (d->heads > 1 && d->stride_h == 0) return LITE_ATTN_EINVAL;
  if (d->head_dim != 128 || d->tile_q != 128 || d->tile_k != 128) return LITE_ATTN_EUNSUPPORTED;
  const int64_t Tk = ((int64_t)d->seqlen + 127) / 128;
  // LDS budgets: the row schedule's histogram (Tk + 1 bins) and the fused kernel's bitmap of newly set mask bits
  if (Tk > 16383) return LITE_ATTN_EUNSUPPORTED;
  // K/V stages are addressed with 32-bit byte offsets from the head's base pointer
  if (((int64_t)d->seqlen + 128) * d->stride_n * 2 >= ((int64_t)1 << 32)) return LITE_ATTN_EUNSUPPORTED;
  const int64_t rows = (int64_t)d->batch * d->heads * Tk;
  if (rows > (int64_t)1 << 30) return LITE_ATTN_EUNSUPPORTED;
  return LITE_ATTN_OK;
}

int check_call(const void* q, const void* k, const void* v, const void* out, float threshold) {
  if (!q || !k || !v || !out) return LITE_ATTN_EINVAL;
  if (std::isnan(threshold) || threshold >= 0.f) return LITE_ATTN_EINVAL;
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out) & 15) return LITE_ATTN_EINVAL;
  return LITE_ATTN_OK;
}

namespace {
size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Partial results of rows cut into segments: what the fused kernel hands to the merge pass.
size_t segment_bytes(const Geometry& g, int nseg) {
  return nseg > 1 ? sizeof(float) * (size_t)g.rows * (nseg * (128 * 128 + 2 * 128) + (size_t)g.Tk * 128) : 0;
}

// How few rows share the chip: how many segments (workgroups) a row is cut into, and whether a workgroup is a pair of
// groups of four waves that take a column half of every tile each.  The chip holds 512 workgroups of four waves, two
// per CU, or 256 pairs.  A CU with a single wave per SIMD takes 1.69 us for a tile (a wave's instructions issue one after
// the other: 2050 cycles for a stage of 1024 matrix cycles), a pair 1.36 us and 2.7 us more per row for its merge in
// LDS, two workgroups on a CU 2.7 us for a tile each, a further round of workgroups 5 us.  Cutting a row costs a second
// launch, 64 KB of fp32 partials per segment written and read again, and the walk over the tiles' row maxima in the merge
// pass (3 us, 0.8 us per four segments, 18 ns per segment, 30 ns per row and 0.15 us per tile of a segment).  Minimum of a
// cost in units of 10 ns made of these measurements.  They fit calls of 3..300 rows with an earlier, slower merge pass and
// while the exponents' reference trailed the maximum (since it follows it again a tile takes 1.88 us, in a pair 1.53, at the
// same ratio).  With both as they are, every number of segments, with and without pairs, of 27 shapes between 3 x 1 and
// 300 x 60 timed on a dense step: the choice is the best of all or within 5 % of it, and within 7 % at 155 x 31 (54.0 in
// pairs, 50.6 in 3 segments).  us per call, whole rows -> segments: 32 rows of 16 tiles 33.0 -> 18.1 (8 segments; 6 17.5),
// 72 x 12 26.6 -> 22.1 (3), 100 x 100 180 -> 84.9 (5); -> pairs: 256 x 64 130 -> 121, 135 x 15 32.8 -> 30.3; -> both: 64 x 64
// 117 -> 44.6 (4; 8 single groups 43.5), 128 x 128 228 -> 129 (2).  The immediate variant needs a tile's verdict before its PV
// product, which a segment cannot know: never cut.
void share_chip(Geometry& g, int flags) {
  const int most = (flags & LITE_ATTN_PV_SKIP_IMMEDIATE) ? 1 : std::min(kMaxSegments, g.Tk);
  int64_t best = -1;
  for (int s = 1; s <= most && (s == 1 || segment_bytes(g, s) <= kMaxSegmentBytes); ++s) {
    const int64_t wgs = g.rows * s, tiles = (g.Tk + s - 1) / s, full = wgs / 512, last = wgs % 512;
    const int64_t merge = s > 1 ? 300 + 80 * ((s + 3) / 4) + 18 * wgs / 10 + 3 * g.rows + 15 * tiles : 0;
    for (int pair = 0; pair < (wgs <= kPairWorkgroups ? 2 : 1); ++pair) {
      const int64_t tile = pair ? 136 : 270 * full + (last == 0 ? 0 : last <= 256 ? 169 : 270);
      const int64_t cost = merge + tiles * tile + (pair ? 270 : 500 * (full + (last != 0) - 1));
      if (best < 0 || cost < best) {
        best = cost;
        g.nseg = s;
        g.pair = pair;
      }
    }
  }
}

// Partial results and row maxima of rows cut into pieces.  (For no layer more than kMaxSegmentBytes, nor with the lists
// more than LITE_ATTN_STATIC_SCRATCH_BYTES: few rows have few tiles each, and of more rows only those beyond whole
// rounds are cut.)
size_t piece_count(const Geometry& g) {
  return g.rows > kFewRows ? 8 * (size_t)cut_rows(g) * cut_pieces(g) : std::max<size_t>(g.pieces, g.rows * equal_pieces(g));
}
size_t piece_bytes(const Geometry& g) {
  const size_t rows = g.rows > kFewRows ? 8 * (size_t)cut_rows(g) : (size_t)g.rows;  // that have row maxima to keep
  return g.pieces > 0 ? sizeof(float) * (piece_count(g) * (128 * 128 + 2 * 128) + rows * g.Tk * 128) : 0;
}

// More rows than run side by side: at an empty mask all are of one length, and the rows beyond whole rounds of
// workgroups would take a round of their own with most of the chip idle, so they are cut, into the more pieces the
// fewer they are; not where they nearly fill it, and not into pieces of fewer than six tiles (a piece costs about two
// tiles' time besides its own).  us, step 0, whole -> cut: 522 rows x 58 tiles 311 -> 251 (4 pieces), 600 x 60 335 ->
// 287 (4), 800 x 40 277 -> 266 (3), 1100 x 55 500 -> 460 (4), 1308 x 110 1087 -> 1034 (3), 1600 x 50 628 -> 600 (4),
// 896 x 128 893 -> 858 (2), 868 x 62 455 -> 442 (2), 870 x 145 1023 -> 983 (2), 1386 x 66 742 -> 717 (2), 1350 x 150
// 1618 -> 1542 (2); no gain in two pieces at 2384 x 150 (2529 -> 2532).  Under a mask rows stay whole (cut
// alike, 800 x 40 at 40 % skipped was 8 % slower).  Where the host does not know whether the mask is empty, the row
// schedule tells, so that a call's result depends on its inputs and its mask, not on how the caller came by them.
void cut_last_round(Geometry& g) {
  const int rest = (int)(g.rows % kFewRows);
  const int each = rest <= 128 ? 4 : rest <= 320 ? 3 : rest <= 400 && g.Tk >= 60 && g.rows < 3 * kFewRows ? 2 : 1;
  if (rest == 0 || each == 1 || g.Tk < 6 * each) return;
  g.pieces = (rest + 7) / 8 << 4 | each;
}
static_assert(400 / 8 <= kArrivals, "a counter for every row that is cut");
static_assert(6 * 3 >= kDrawTiles, "calls that cut rows clear their counters");

// Few rows: whether calls that mark cut the rows by their live tiles (pick_piece() in lite_attn_kernels.hip) instead of
// all alike: into at most as many pieces as the chip runs side by side, pairs or, with more rows, single groups.  us
// per call of a sequence of 3-4 steps (the first is dense), alike -> by live tiles: whole rows, 135 x 15 tiles 31.8 ->
// 28.7, 155 x 31 56 -> 46.6, 290 x 29 90.9 -> 71.5, 300 x 10 38.3 -> 36.3; segments and merge pass, 100 x 25 34.0 ->
// 30.8, 128 x 64 66.4 -> 62.2, 99 x 99 80.6 -> 73.7, 300 x 60 137.5 -> 124.1.  Not where the room is taken by the rows
// themselves (184 of 256 -3 %, 250 -2 %), nor where a row has so few tiles that finding the pieces (1-2 us) costs what
// it saves (128 x 8 -11 %, 72 x 12 in segments -10 %) or so many segments that more than kMaxPieces would be needed (64
// x 32 -1 %).  The literal PV skip can only cut rows of protected tokens, whose tiles need no verdict; diagonal first
// they are the only long ones (155 x 31, 10 of them protected, four steps 247 -> 155 us; in ascending order -2 %).
// Rows that a mask has left alike gain nothing and pay 1-2 us.  The allocation-free call, which has nobody to count for
// it, pays a launch more, 2.5 us, even at an empty mask: us, before there were pieces -> now, empty / 40 % of each row's
// tiles skipped / rows of 0 to 100 %, 155 x 31 56.2 -> 58.1 / 45.1 -> 40.4 / 54.1 -> 40.0, 135 x 15 31.1 -> 33.4 / 26.9 ->
// 26.5 / 30.3 -> 24.6, 300 x 10 38.8 -> 40.5 / 31.2 -> 32.5 / 33.9 -> 31.7.
void allow_pieces(Geometry& g, const lite_attn_desc_t& d) {
  const bool immediate = (d.flags & LITE_ATTN_PV_SKIP_IMMEDIATE) != 0;
  if (immediate && (d.protect_len == 0 || !(d.flags & LITE_ATTN_ORDER_DIAGONAL_FIRST))) return;
  if (g.nseg > 1 ? g.Tk < 16 || g.rows < 80 : g.Tk < 10) return;
  const bool pairs = g.nseg > 1 ? 10 * g.rows <= 7 * kPairWorkgroups : g.pair != 0;
  const int room = pairs ? kPairWorkgroups : kFewRows;
  if (10 * g.rows > 7 * room) return;
  g.pieces = room;
}
}  // namespace

// Few rows that may be cut into pieces: how many of each a call that marks makes where the mask is empty, whether the
// caller knows it (segments and merge pass) or the counts say so (pieces; the same sums in the same order).  As many as
// share_chip() finds, if that is for the same kind of workgroups; else as many as fill one round of pairs, or, with
// more than half as many rows as that, three in two rounds.  us, step 0, share_chip()'s single groups -> pairs: 80 x 20
// 27.9 -> 27.3, 100 x 25 39.4 -> 36.3, 105 x 35 46.4 -> 46.1, 128 x 64 80.4 -> 80.8, 99 x 99 96.3 -> 102.1, 130 x 65
// 90.4 -> 101.8, 150 x 150 199.8 -> 211.3 (with today's merge pass, 100 x 100 89.5 -> 97.2, 130 x 65 82.3 -> 92.7): what it
// costs that a mask's pieces are pairs, and that a call's result depends on its inputs and its mask, not on how the caller
// came by them.
int equal_pieces(const Geometry& g) {
  if (g.rows > kFewRows) return 1;
  if (g.nseg == 1 || (g.pieces == kPairWorkgroups) == (g.pair != 0)) return g.nseg;
  const int rows = (int)g.rows;
  return 2 * rows <= kPairWorkgroups ? kPairWorkgroups / rows : 3 * rows <= 2 * kPairWorkgroups ? 3 : 1;
}

Geometry geometry(const lite_attn_desc_t& d) {
  Geometry g;
  g.Tq = (d.seqlen + d.tile_q - 1) / d.tile_q;
  g.Tk = (d.seqlen + d.tile_k - 1) / d.tile_k;
  g.W = (g.Tk + 63) / 64;
  g.run_stride = g.Tk / 2 + 1;
  g.BH = d.batch * d.heads;
  g.rows = (int64_t)g.BH * g.Tq;
  g.chunks = g.BH * ((g.Tq + kChunkRows - 1) / kChunkRows);
  g.nseg = 0;
  g.pair = 0;
  g.pieces = 0;
  g.per_xcd = ((g.chunks + 7) / 8 + 1) * kChunkRows + 1;
  if (g.rows <= kFewRows || (g.Tk <= kShortTiles && g.rows <= kMaxListless)) {
    g.nseg = 1;
    if (g.rows <= kFewRows) {
      share_chip(g, d.flags);
      allow_pieces(g, d);
    } else if (g.rows <= kSchedRows && !(d.flags & LITE_ATTN_PV_SKIP_IMMEDIATE)) {
      cut_last_round(g);
    }
    g.per_xcd = (int)((g.rows * g.nseg + 7) / 8);
    if (g.rows > kSchedRows)
      g.per_xcd = (int)((g.rows + 8 * kDealtRows - 1) / (8 * kDealtRows)) * kDealtRows;
    else if (g.rows > kFewRows)
      g.per_xcd += g.per_xcd / 2 + kTableTail;  // room for an XCD whose rows are short
  }
  return g;
}

// A row schedule is an order of the rows, good for any mask; when later calls have marked some more tiles, the lengths it
// was made for are a little off.
bool keeps_table(const Geometry& g) { return g.nseg > 0 && g.rows > kFewRows && g.rows <= kSchedRows; }

ListLayout list_layout(const Geometry& g) {
  ListLayout l;
  size_t at = 0;
  l.nruns = at;
  at += up256(sizeof(uint32_t) * (size_t)g.rows);
  l.live_cnt = at;
  at += up256(sizeof(uint32_t) * (size_t)g.rows);
  l.order = at;
  if (g.nseg == 0) at += up256(sizeof(uint32_t) * (size_t)g.rows);
  l.chunk_work = at;
  if (g.nseg == 0) at += up256(sizeof(uint32_t) * (size_t)g.chunks);
  l.slots = at;
  at += up256(sizeof(uint32_t) * 8 * (size_t)g.per_xcd);
  l.xcd_rows = at;
  l.heads_ranked = at + sizeof(uint32_t) * 8;
  at += up256(sizeof(uint32_t) * 9);
  l.tickets = l.slots;
  if (keeps_table(g)) {
    l.tickets = at;
    at += up256(sizeof(uint32_t) * 8 * (kTicketWords + kArrivals));
  }
  l.runs = at;
  at += up256(sizeof(uint32_t) * (size_t)g.rows * g.run_stride);
  l.total = at;
  return l;
}

ScratchLayout scratch_layout(const Geometry& g, int nseg) {
  const size_t parts = nseg > 1 ? (size_t)g.rows * nseg : piece_count(g);
  ScratchLayout l;
  l.seg_o = 0;
  l.seg_stat = sizeof(float) * parts * 128 * 128;
  l.seg_mloc = l.seg_stat + sizeof(float) * parts * 2 * 128;
  l.total = up256(g.nseg > 0 ? std::max(segment_bytes(g, g.nseg), piece_bytes(g))
                             : sizeof(uint16_t) * (size_t)g.BH * 128 * ((size_t)g.Tk * 128));
  return l;
}

}  // namespace la
