// TEST INFRASTRUCTURE (see hip/hip_runtime.h next to this file): host stand-ins for the kernel launchers.  They compute
// nothing of the method; each one writes every byte its kernel is entitled to write, so that AddressSanitizer sees
// whether the host code handed it buffers of the right size (scratch layout, mask and statistics allocations).  Schedules
// hold a real permutation of the rows, and an attention launch checks that the one it is given does; calls that can mark set
// a bit of every row.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <vector>

#include "lite_attn_kernels.h"

unsigned long long fake_capture = 0;

namespace {

std::vector<std::vector<std::function<hipError_t()>>> graphs;  // graph x: the launches of capture x + 1

// A launch: made at once, or kept for the replays of the capture under way on its stream.
template <class F>
hipError_t launch(hipStream_t st, F f) {
  if (!st || !fake_capture) return f();
  graphs.back().push_back(f);
  return hipSuccess;
}

// Pieces of one allocation that must not run into the piece behind them (AddressSanitizer sees only the allocation's end).
bool before(const void* end, const void* next) { return (uintptr_t)end <= (uintptr_t)next; }

// All rows, dealt to the XCDs in turn; no entry of the table but these is a row.
void deal(uint32_t* slots, int per_xcd, uint32_t* xcd_rows, int rows) {
  memset(slots, 0xff, sizeof(uint32_t) * 8 * (size_t)per_xcd);  // the whole table may be written
  for (int x = 0; x < 8; ++x) {
    xcd_rows[x] = 0;
    for (int r = x; r < rows; r += 8) slots[(size_t)x * per_xcd + xcd_rows[x]++] = (uint32_t)r;
  }
}

bool every_row_once(const uint32_t* slots, int per_xcd, const uint32_t* xcd_rows, int rows) {
  std::vector<char> seen(rows);
  for (int x = 0; x < 8; ++x)
    for (uint32_t t = 0; t < xcd_rows[x]; ++t) {
      if (t >= (uint32_t)per_xcd) return false;
      const uint32_t r = slots[(size_t)x * per_xcd + t];
      if (r == 0xffffffffu) continue;
      if (r >= (uint32_t)rows || seen[r]++) return false;
    }
  return std::count(seen.begin(), seen.end(), 1) == rows;
}

// Lists: one run covering the row, [0, Tk), whatever the mask; the live tiles tell whether its first tile is marked.
uint32_t live_tiles(const uint64_t* bits, int r, int Tk, int W) { return (uint32_t)Tk - (uint32_t)(bits[(size_t)r * W] & 1); }
void lists_of(const uint64_t* bits, int rows, int Tk, int W, int run_stride, uint32_t* runs, uint32_t* nruns,
              uint32_t* live_cnt) {
  for (int r = 0; r < rows; ++r) {
    memset(runs + (size_t)r * run_stride, 0, sizeof(uint32_t) * run_stride);
    runs[(size_t)r * run_stride] = (uint32_t)Tk << 16;
    nruns[r] = 1;
    live_cnt[r] = live_tiles(bits, r, Tk, W);
  }
}

bool all_zero(const uint64_t* bits, size_t words) { return std::count(bits, bits + words, 0) == (long)words; }

}  // namespace

extern "C" {
void fake_begin_capture() {
  graphs.emplace_back();
  fake_capture = graphs.size();
}
int fake_end_capture() {
  fake_capture = 0;
  return (int)graphs.size();
}
int fake_replay(int graph) {
  for (auto& f : graphs[graph - 1])
    if (const hipError_t e = f()) return e;
  return 0;
}
}

namespace la {

hipError_t prepare_fwd() { return hipSuccess; }

static hipError_t clear(uint64_t* bits, size_t words, unsigned long long* stats, size_t nstats) {
  if (words) memset(bits, 0, words * sizeof(uint64_t));
  if (nstats) memset(stats, 0, nstats * sizeof(unsigned long long));
  return hipSuccess;
}
hipError_t launch_clear(uint64_t* bits, size_t words, unsigned long long* stats, size_t nstats, hipStream_t st) {
  return launch(st, [=] { return clear(bits, words, stats, nstats); });
}

static hipError_t count_rows(const uint64_t* bits, int rows, int W, uint32_t* live, uint32_t* arrive) {
  const bool empty = all_zero(bits, (size_t)rows * W);
  for (int r = 0; r < rows; ++r) live[r] = empty ? 0 : 1;
  if (arrive) memset(arrive, 0, sizeof(uint32_t) * rows);
  return hipSuccess;
}
hipError_t launch_count_rows(const uint64_t* bits, int rows, int, int W, uint32_t* live, uint32_t* arrive, hipStream_t st) {
  return launch(st, [=] { return count_rows(bits, rows, W, live, arrive); });
}

static hipError_t compact(const uint64_t* bits, int rows, int Tk, int W, int run_stride, uint32_t* runs, uint32_t* nruns,
                          uint32_t* live_cnt, uint32_t* heads_ranked) {
  *heads_ranked = 0;
  lists_of(bits, rows, Tk, W, run_stride, runs, nruns, live_cnt);
  return hipSuccess;
}
hipError_t launch_compact(const uint64_t* bits, int rows, int, int Tk, int W, int, int run_stride, uint32_t* runs,
                          uint32_t* nruns, uint32_t* live_cnt, uint32_t* heads_ranked, hipStream_t st) {
  return launch(st, [=] { return compact(bits, rows, Tk, W, run_stride, runs, nruns, live_cnt, heads_ranked); });
}

static hipError_t clear_tickets(uint32_t* tickets, int stride) {
  for (int x = 0; x < 8; ++x) tickets[(size_t)x * stride] = 0;
  return hipSuccess;
}
hipError_t launch_clear_tickets(uint32_t* tickets, int stride, hipStream_t st) {
  return launch(st, [=] { return clear_tickets(tickets, stride); });
}

static hipError_t prepare_rows(const RowSchedule& p, uint16_t* vt) {
  if (*p.heads_ranked != 0) return hipErrorInvalidValue;  // zero between launches
  for (int x = 0; x < p.BH * p.Tq; ++x) p.order[x] = p.live_cnt[x] ? (uint32_t)(x % p.Tq) : 0u;
  for (int u = 0; u < p.chunks; ++u) p.chunk_work[u] = 1;
  if (!before(p.slots + 8 * (size_t)p.per_xcd, p.xcd_rows)) return hipErrorInvalidValue;
  deal(p.slots, p.per_xcd, p.xcd_rows, p.BH * p.Tq);
  clear_tickets(p.slots + p.per_xcd - 1, p.per_xcd);
  memset(vt, 0, sizeof(uint16_t) * (size_t)p.BH * 128 * ((size_t)p.Tk * 128));
  return hipSuccess;
}
hipError_t launch_prepare_rows(const RowSchedule& p, const uint16_t*, uint16_t* vt, int64_t, int64_t, int64_t, int, int,
                               hipStream_t st) {
  return launch(st, [=] { return prepare_rows(p, vt); });
}

static hipError_t schedule_rows(const uint64_t* bits, int rows, int W, int per_xcd, uint32_t* slots, uint32_t* xcd_rows) {
  if (!before(slots + 8 * (size_t)per_xcd, xcd_rows)) return hipErrorInvalidValue;
  deal(slots, per_xcd, xcd_rows, rows);
  for (int x = 1; x <= 8; ++x) {  // flag, marks, arrivals, ticket
    memset(slots + (size_t)x * per_xcd - kTableTail, 0, sizeof(uint32_t) * kTableTail);
    slots[(size_t)x * per_xcd - kTableTail] = all_zero(bits, (size_t)rows * W);
  }
  return hipSuccess;
}
hipError_t launch_schedule_rows(const uint64_t* bits, int rows, int, int W, int per_xcd, uint32_t* slots,
                                uint32_t* xcd_rows, hipStream_t st) {
  return launch(st, [=] { return schedule_rows(bits, rows, W, per_xcd, slots, xcd_rows); });
}

namespace {

// Partial results of `parts` segments or pieces and the row maxima of `rows` rows, each before the next.
bool partials(const FwdParams& p, size_t parts, size_t rows) {
  if (!before(p.seg_o + parts * 128 * 128, p.seg_stat) || !before(p.seg_stat + parts * 2 * 128, p.seg_mloc)) return false;
  memset(p.seg_o, 0, sizeof(float) * parts * 128 * 128);
  memset(p.seg_stat, 0, sizeof(float) * parts * 2 * 128);
  memset(p.seg_mloc, 0, sizeof(float) * rows * p.Tk * 128);
  return true;
}

// Few or short rows: no lists and no V^T.  Rows that several workgroups share leave partial results in the scratch; rows beyond
// the first round are drawn; at step 0 the mask is overwritten and, with few rows, all counters are cleared.
hipError_t fwd_without_lists(const FwdParams& p) {
  const size_t rows = (size_t)p.rows_total;
  if (p.scheduled && !every_row_once(p.slots, p.per_xcd, p.xcd_rows, p.rows_total)) return hipErrorInvalidValue;
  // what lies behind the tickets and the arrival counters of a call: the end of its table, or of those that have no table
  const uint32_t* behind = p.tickets > p.xcd_rows ? p.runs : p.xcd_rows;
  if (p.tickets && p.resident == kResident)  // counters start at zero
    for (int x = 0; x < 8; ++x)
      if (!before(p.tickets + x * p.ticket_stride + 1, behind) || p.tickets[x * p.ticket_stride]++ != 0)
        return hipErrorInvalidValue;
  if (p.nseg > 1 && !partials(p, rows * p.nseg, rows)) return hipErrorInvalidValue;
  if (p.piece_units > 0) {
    if (!partials(p, std::max<size_t>(p.piece_units, rows * p.equal_pieces), rows)) return hipErrorInvalidValue;
    for (size_t r = 0; r < rows; ++r)  // arrivals start at zero and are zero again behind the call
      if (p.arrive[r] != 0 || (int)p.live_rows[r] > p.Tk) return hipErrorInvalidValue;
  }
  if (p.cut_rows > 0) {
    if (p.scheduled) {  // rows are cut if, and only if, the mask is empty, which the table and its calls' marks tell
      bool empty = p.slots[(size_t)p.per_xcd - kTableTail] != 0;
      for (int x = 0; x < p.table_calls; ++x) empty = empty && !p.marked[x];
      if (empty != all_zero(p.bits, rows * p.W)) return hipErrorInvalidValue;
    }
    const size_t cut = 8 * (size_t)p.cut_rows;
    if (!partials(p, cut * p.cut_pieces, cut)) return hipErrorInvalidValue;
    for (int x = 0; x < 8; ++x)
      for (int r = 0; r < p.cut_rows; ++r) {
        uint32_t* at = p.arrive + x * p.arrive_stride + r;
        // (not the ticket, which the loop above has moved)
        if (!before(at + 1, behind) || *at != 0) return hipErrorInvalidValue;
      }
  }
  if (p.fresh && p.newly_rows) {
    memset(p.stats_all, 0, sizeof(unsigned long long) * (size_t)p.stat_words);
    memset(p.newly_rows, 0, sizeof(uint32_t) * rows);
  }
  if (p.live_next) {
    if (p.piece_units > 0 && p.live_next == p.live_rows) return hipErrorInvalidValue;  // (read while it is written)
    for (size_t r = 0; r < rows; ++r) p.live_next[r] = (uint32_t)p.Tk;
  }
  if (p.fresh) memset(p.bits, 0, sizeof(uint64_t) * rows * p.W);
  return hipSuccess;
}

}  // namespace

static hipError_t fwd(const FwdParams& p) {
  const size_t rows = (size_t)p.rows_total;
  if (p.nseg > 0) {
    const hipError_t e = fwd_without_lists(p);
    if (e != hipSuccess) return e;
  } else {
    // the first and last element of everything the kernel reads or writes besides q, k, v, out
    volatile uint32_t sink = p.runs[0] + p.runs[rows * p.run_stride - 1] + p.nruns[rows - 1] + p.live_cnt[rows - 1] +
                             p.vt[(size_t)(rows / p.Tq) * 128 * ((size_t)p.Tk * 128) - 1];
    (void)sink;
    if (!every_row_once(p.slots, p.per_xcd, p.xcd_rows, p.rows_total)) return hipErrorInvalidValue;
    for (int x = 0; x < 8; ++x)
      if (p.tickets && p.tickets[x * p.ticket_stride]++ != 0) return hipErrorInvalidValue;
    for (size_t r = 0; r < rows; ++r)  // the lists are those of the mask
      if (p.nruns[r] != 1 || p.live_cnt[r] != live_tiles(p.bits, (int)r, p.Tk, p.W)) return hipErrorInvalidValue;
  }
  for (size_t r = 0; p.thr > -INFINITY && r < rows; ++r) {
    *p.stat_newly += !(p.bits[r * p.W] & 1);
    if (p.marked && !(p.bits[r * p.W] & 1)) p.marked[p.table_calls] = 1;
    p.bits[r * p.W] |= 1;
  }
  if (p.build_next && p.nseg == 0)  // the epilogue rewrites the lists in full
    lists_of(p.bits, p.rows_total, p.Tk, p.W, p.run_stride, p.runs, p.nruns, p.live_cnt);
  *p.stat_skipped_in += 0;
  *p.stat_runs += (unsigned long long)rows;
  return hipSuccess;
}
hipError_t launch_fwd(const FwdParams& p, bool, hipStream_t st) {
  return launch(st, [=] { return fwd(p); });
}

}  // namespace la
