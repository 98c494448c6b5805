// Internal interface between the C-ABI host code and the gfx950 kernels (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "lite_attn.h"

namespace la {

// Rows of one head that an XCD runs side by side (2 workgroups x 32 CUs): the unit of the row schedule ("chunk").
constexpr int kChunkRows = 64;

// Calls with few rows or short rows take no Skip-Lists and no V^T (template argument FEW; measurements at
// schedule_rows_kernel): at most kFewRows Q-tile rows -- all of whose workgroups fit the chip at once; they need no schedule
// and may be cut into segments, whose partial results stay small enough for the static scratch array -- or at most
// kShortTiles tiles a row.  Beyond kSchedRows rows there are so many rounds of workgroups that the order of the rows inside
// an XCD does not matter and no table is made: chunks of kDealtRows rows go to the XCDs in turn (dealt_chunk).
constexpr int kFewRows = 512;
constexpr int kShortTiles = 192;
constexpr int kMaxListless = 1 << 23;  // rows; the kernel's short division and its grid hold for that many
constexpr int kSchedRows = 32768;
constexpr int kDealtRows = kChunkRows;
// Workgroups that an XCD holds at once (two per CU): the first round takes the rows that its place in the grid names, later
// workgroups draw theirs (FwdParams::tickets).
constexpr int kResident = 64;
constexpr int kNoDraws = 1 << 30;
// Rows of fewer tiles than this go by place alone.  us, drawn (and a workgroup for every entry of the table's tail) ->
// by place: a later step of 1000 rows of 1 tile 38.4 -> 28.3, 4000 x 1 123 -> 96, 2000 x 2 71 -> 55, 4900 x 7 278 ->
// 258, 33001 x 1 714 -> 629, 80000 x 4 2834 -> 2688; 36000 x 12 2527 -> 2505; drawn / by place, without the tail's
// workgroups: 1200 x 12 90.2 / 89.8, 12000 x 12 1001 / 988, 8000 x 16 822 / 835, 33600 x 16 2926 / 2946, 7200 x 24 1039
// / 1059, 33600 x 24 4105 / 4167.
constexpr int kDrawTiles = 16;
constexpr int kTicketWords = 32;  // distance of the counters of an unscheduled call, a cache line
constexpr int kArrivals = 64;     // arrival counters per XCD, of rows cut alike (cut_rows)
constexpr int kTableCalls = 8;    // calls that a row schedule serves (keeps_table)
// End of an XCD's share of a short rows' table: a flag, marks of the table's calls (XCD 0's are used), arrivals, the ticket.
constexpr int kTableTail = 2 + kTableCalls + kArrivals;
constexpr int kPairWorkgroups = 256;
constexpr int kClearWords = 64;   // us, 3 rows x 1 tile, 64 for each thread 9.6 (a launch: 8.9), 4096 for each 174 (12.1)
constexpr int kMaxSegments = 16;
// Pieces of a row that a mask asks for.  us, four steps, at most 2 / 3 / 4 / 8: 100 x 25 140 / 125 / 123 / 123, 105 x 35
// 173 / 149 / 146 / 146, 99 x 99 364 / 307 / 285 / 286, 300 x 60 495 / 481 / 480 / 480; literal skip, whose protected
// rows alone are long, 155 x 31 192 / 169 / 157 / 152, 126 x 63 329 / 275 / 251 / 242.
constexpr int kMaxPieces = 4;
constexpr size_t kMaxSegmentBytes = (size_t)104 << 20;

// The chunk of rows that XCD `xcd` takes of the `group`-th eight chunks.  The assignment turns from group to group, in
// three periods, so that heads that differ with a period of their own (the heads of a layer, batch entry after batch entry)
// do not all fall to one XCD.
constexpr int dealt_chunk(int group, int xcd) { return 8 * group + ((xcd - group - group / 8 - group / 64) & 7); }

struct FwdParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* vt;                    // V^T scratch: [B*H][128][128*Tk], written by launch_prepare_rows
  uint16_t* out;
  int64_t stride_b, stride_h, stride_n;  // elements
  int H, N, Tq, Tk, W;                   // W = uint64 words per mask row
  uint32_t* runs;                        // [rows][run_stride] Skip-List: start | end << 16 per run of live tiles
  int run_stride;
  uint32_t* nruns;                       // [rows] runs per row
  uint32_t* live_cnt;                    // [rows] live tiles per row
  uint64_t* bits;                        // [rows][W]
  unsigned long long* stat_skipped_in;   // counters of the current step
  unsigned long long* stat_newly;
  unsigned long long* stat_runs;
  float thr;                             // signed threshold, natural-log units of S
  float scale;                           // 1/sqrt(d)
  int protect_start, protect_len;
  int rows_total;                        // B*H*Tq
  const uint32_t* slots;                 // [8][per_xcd]: the row (index into [B*H][Tq]) that workgroup `slot` of an
  int per_xcd;                           //   XCD computes, written by launch_prepare_rows; entries >= xcd_rows[xcd] unused
  const uint32_t* xcd_rows;              // [8] rows dealt to each XCD
  uint32_t* tickets;                     // [8] at ticket_stride: rows drawn so far from each XCD's list beyond the first
  int ticket_stride;                     //   `resident`; null: few rows, each workgroup has its place
  int table_calls = 0;                   // calls that the table has served before this one
  uint32_t* marked = nullptr;            // cut_rows > 0, scheduled: [kTableCalls] whether the table's calls have marked a tile,
                                         //   by call; a call looks at those before it
  int resident;                          // places per XCD that go by the grid: kResident, or, where rows are too short to be
                                         //   drawn, kNoDraws
  // build_next != 0: the epilogue rewrites runs / nruns / live_cnt for the NEXT call from the mask this call leaves;
  // diagonal_first: visiting order of the lists
  int build_next, diagonal_first;
  // Few or short rows (nseg > 0, see Geometry): V read as it is, the row's live tiles found from its mask row, no lists;
  // the row cut into nseg segments, one workgroup each.
  int nseg = 0;
  int pair = 0;
  // Not scheduled: the (head, segment, row) triples in order, an eighth of them to each XCD; beyond kSchedRows rows chunks.
  int scheduled = 0;
  int fresh = 0;                         // step 0: the mask counts as empty and is overwritten
  const uint16_t* v = nullptr;
  float* seg_o = nullptr;                // [rows][nseg][128][128] O^T partials in accumulator order
  float* seg_stat = nullptr;             // [rows][nseg][2][128]: row maximum (the exponents' reference), row sum
  float* seg_mloc = nullptr;             // [rows][Tk][128]: row maxima of the visited tiles
  unsigned long long* stats_all = nullptr;  // all counters of the handle (stat_words of them)
  int64_t stat_words = 0;
  // > 0: the rows are cut into pieces by their live tiles, at most this many altogether (pick_piece).  Their partial
  // results are in seg_o and seg_stat, by piece, the row maxima in seg_mloc.
  int piece_units = 0;
  int equal_pieces = 1;                  //   where their lengths do not ask for another cut: into this many each
  int alike = 0;                         //   (which the caller knows: alike != 0)
  int cut_rows = 0, cut_pieces = 1;      // more than kFewRows rows: of each eighth, by number, the last cut_rows are
                                         //   cut alike if the mask is empty (no schedule, or its flag says so)
  uint32_t* arrive = nullptr;            // pieces that have arrived: [rows], zero between calls, or [8] at arrive_stride
  int arrive_stride = 0;                 //   [cut_rows], cleared by the schedule or clearing kernel
  const uint32_t* live_rows = nullptr;   // piece_units > 0: [rows] live tiles, counted before the launch
  uint32_t* live_next = nullptr;         // [rows] live tiles that this call leaves, for the next one; may be null
  uint32_t* newly_rows = nullptr;        // few rows: [rows] tiles that step 0 marks (the kernel clears the counters)
  int parts = 1;                         // nseg * equal_pieces
  uint32_t per_Tq, per_H, per_parts = 0;  // reciprocals for the kernel's short division
};

// a / b (a >= 0, b >= 1, a + b < 2^31) with the host's per_b = reciprocal(b): a * per_b / 2^32 is short of a / b by less
// than one.  On the GPU a few scalar instructions; a workgroup with few tiles waits for its indexes before its first load.
constexpr uint32_t reciprocal(int b) { return b == 1 ? 0xffffffffu : (uint32_t)(((uint64_t)1 << 32) / (uint32_t)b); }
constexpr int quotient(int a, int b, uint32_t per_b) {
  const int q = (int)((uint64_t)(uint32_t)a * per_b >> 32);
  return (q + 1) * b <= a ? q + 1 : q;
}

// Tile geometry of a layer, derived from its descriptor.
struct Geometry {
  int Tq, Tk, W;   // Q tiles, K/V tiles, uint64 words per Skip-Mask row
  int run_stride;  // capacity of one row's run-length Skip-List: floor(Tk/2) + 1 runs (ascending order needs at most
                   // ceil(Tk/2); diagonal first can split one more run at the wrap-around)
  int BH;          // batch * heads
  int pieces;      // > 0: few rows, cut by their live tiles into at most this many pieces (workgroups; pairs, if it is
                   // kPairWorkgroups), or, at an empty mask, into equal_pieces() each; nseg and pair are then for calls that
                   // mark nothing.  Beyond kFewRows rows: how some of them are cut (cut_rows, cut_pieces)
  int64_t rows;    // BH * Tq
  int chunks;      // BH * ceil(Tq / kChunkRows): units of the row schedule
  int pair;        // workgroups of two groups of four waves (at most kPairWorkgroups of them)
  int nseg;        // > 0: few or short rows, each cut into this many segments (one workgroup each; 1 beyond kFewRows rows);
                   // 0: Skip-Lists, row ranking and V^T
  int per_xcd;     // entries per XCD in the schedule table: row slots, with lists (ceil(chunks / 8) + 1) chunks, short rows
                   // 1.5 shares and kTableTail words; where there is no table, the workgroups of an XCD
};

// More than kFewRows rows: rows of each eighth, by number, that are cut, and into how many pieces each.
constexpr int cut_rows(const Geometry& g) { return g.rows > kFewRows ? g.pieces >> 4 : 0; }
constexpr int cut_pieces(const Geometry& g) { return g.rows > kFewRows ? g.pieces & 15 : 0; }

// Byte offsets of the Skip-List buffers inside one allocation (256-byte aligned pieces).  Handles keep them between
// calls (a call's epilogue leaves the next call's lists there); the handle-free entry point rebuilds them per call.
struct ListLayout {
  size_t nruns;     // [rows] uint32 runs per row
  size_t live_cnt;  // [rows] uint32 live tiles per row
  size_t order;     // [BH][Tq] uint32 row ranking (none with few or short rows)
  size_t chunk_work;  // [chunks] uint32 work of each chunk (live tiles + a per-row constant)
  size_t slots;     // [8][per_xcd] uint32 schedule table
  size_t xcd_rows;  // [8] uint32
  size_t heads_ranked;  // uint32, a counter of prepare_rows_kernel, zero between launches
  size_t tickets;   // [8] tickets at kTicketWords, [8][kArrivals] arrival counters, of calls that make no table: behind the
                    //   table of layers that also make one, else where it would be
  size_t runs;      // [rows][run_stride] uint32 Skip-List
  size_t total;
};

// lite_attn_host.cpp (no HIP calls): argument checks shared by the entry points, geometry, scratch layout
int check_desc(const lite_attn_desc_t* d);  // LITE_ATTN_OK or the error the header documents
int check_call(const void* q, const void* k, const void* v, const void* out, float threshold);
Geometry geometry(const lite_attn_desc_t& d);
ListLayout list_layout(const Geometry& g);
int equal_pieces(const Geometry& g);
// Scratch of a layer's calls: V^T ([BH][128][128*Tk] bf16), or the partial results of rows cut into nseg segments or,
// at 1, into pieces; rows that stay whole and take no lists need neither (total 0, the most that any of the layer's
// calls needs).
struct ScratchLayout {
  size_t seg_o, seg_stat, seg_mloc, total;
};
ScratchLayout scratch_layout(const Geometry& g, int nseg = 1);

// The row schedule of rows with Skip-Lists, made beside V^T.
struct RowSchedule {
  const uint32_t* live_cnt;
  uint32_t *order, *chunk_work, *slots, *xcd_rows, *heads_ranked;
  int Tq, Tk, BH, chunks, per_xcd;
};

// lite_attn.cpp: the launches of one attention call on `stream`.  lists_ready: the Skip-Lists in `lists` already
// describe the mask (left by the previous call's epilogue); otherwise the compaction kernel builds them first.  Then
// the row schedule, the V^T pre-pass into `scratch` and the fused attention kernel, whose epilogue builds the next call's
// lists if build_next.  With few or short rows (Geometry::nseg > 0) there are no lists and no V^T: the fused kernel, before
// it a schedule or behind it, for rows cut into segments, the merge pass.  `mid` (may be null) is recorded just before the
// attention kernel.  Allocates nothing.
struct CallArgs {
  const void *q, *k, *v;
  void* out;
  float threshold;
  uint64_t* bits;              // the Skip-Mask
  unsigned long long* stats3;  // this step's counters, or null (nobody reads them)
  bool empty;                  // the mask is empty (step 0, or nothing could have marked a tile since): rows are alike
  bool fresh;                  // step 0: the mask counts as empty, whatever it holds, and all counters start at zero
  unsigned long long* stats_all;
  size_t stat_words;
  uint32_t* newly_rows;        // few rows: marks of step 0, per row; null elsewhere
  uint32_t* arrive;            // few rows: kFewRows counters that are zero between calls; null: to be cleared by the call
  const uint32_t* live_rows;   // few rows that may be cut into pieces: live tiles, left by the previous call; null: to
  uint32_t* live_next;         //   be counted.  The same for the next call, or null
  bool lists_ready, build_next;
  int table_calls;             // calls of the trajectory that the row schedule in place has served; 0: to be made
};
// A row schedule of short rows made once and used by several calls: an order of the rows is good for any mask.  us, sixteen
// steps, made by every call / for 4 calls / for 8 / for 16 / once: 888 rows x 37 tiles 3241 / 3168 / 3159 / 3149 / 3149, 640 x
// 16 1223 / 1141 / 1130 / 1123 / 1123, 1320 x 110 6020 / 5979 / 5973 / 5967 / 5985, 2440 x 61 11671 / 11613 / 11602 / 11602 /
// 11613, rows that go by place, 640 x 8 878 / 793 / 781 / 773 / 773, 742 x 14 1277 / 1197 / 1178 / 1167 / 1166; eight steps
// whose inputs have nothing to do with each other, every call / 8, 888 x 37 1613 / 1576, 640 x 16 619 / 581, 1320 x 110 3120 /
// 3065, 2440 x 61 5807 / 5808, 640 x 8 446 / 399, 742 x 14 641 / 597.  The table of rows with lists is made beside V^T and costs
// nothing (600 x 200 and 3072 x 256 0.1 % apart): every call makes its own.
bool keeps_table(const Geometry& g);  // layers that make one

hipError_t launch_call(const lite_attn_desc_t& d, const Geometry& g, const ListLayout& ll, char* lists, char* scratch,
                       const CallArgs& a, hipStream_t stream, hipEvent_t mid);
int hip_fail(hipError_t e);  // remembers e for lite_attn_last_hip_error() and maps it to a lite_attn_error

hipError_t prepare_fwd();
hipError_t launch_clear(uint64_t* bits, size_t words, unsigned long long* stats, size_t nstats, hipStream_t st);
hipError_t launch_count_rows(const uint64_t* bits, int rows, int Tk, int W, uint32_t* live, uint32_t* arrive,
                             hipStream_t st);
hipError_t launch_compact(const uint64_t* bits, int rows, int Tq, int Tk, int W, int diagonal_first, int run_stride,
                          uint32_t* runs, uint32_t* nruns, uint32_t* live_cnt, uint32_t* heads_ranked, hipStream_t st);
hipError_t launch_prepare_rows(const RowSchedule& sched, const uint16_t* v, uint16_t* vt, int64_t stride_b, int64_t stride_h,
                               int64_t stride_n, int H, int N, hipStream_t st);
hipError_t launch_clear_tickets(uint32_t* tickets, int stride, hipStream_t st);
hipError_t launch_schedule_rows(const uint64_t* bits, int rows, int Tk, int W, int per_xcd, uint32_t* slots,
                                uint32_t* xcd_rows, hipStream_t st);
hipError_t launch_fwd(const FwdParams& p, bool immediate, hipStream_t st);

}  // namespace la
