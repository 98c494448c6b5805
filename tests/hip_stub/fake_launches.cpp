// TEST INFRASTRUCTURE (see hip/hip_runtime.h next to this file): host stand-ins for the kernel launchers.  They compute
// nothing of the method; each one writes every byte its kernel is entitled to write, so that AddressSanitizer sees
// whether the host code handed it buffers of the right size (scratch layout, mask and statistics allocations).
#include <string.h>

#include <algorithm>

#include "lite_attn_kernels.h"

namespace {

// Pieces of one allocation that must not run into the piece behind them (AddressSanitizer sees only the allocation's end).
bool before(const void* end, const void* next) { return (uintptr_t)end <= (uintptr_t)next; }

}  // namespace

namespace la {

hipError_t prepare_fwd() { return hipSuccess; }

hipError_t launch_clear(uint64_t* bits, size_t words, unsigned long long* stats, size_t nstats, hipStream_t) {
  if (words) memset(bits, 0, words * sizeof(uint64_t));
  if (nstats) memset(stats, 0, nstats * sizeof(unsigned long long));
  return hipSuccess;
}

hipError_t launch_count_rows(const uint64_t* bits, int rows, int, int W, uint32_t* live, uint32_t* arrive, hipStream_t) {
  uint64_t any = 0;
  for (size_t x = 0; x < (size_t)rows * W; ++x) any |= bits[x];
  for (int r = 0; r < rows; ++r) live[r] = any ? 1 : 0;
  if (arrive) memset(arrive, 0, sizeof(uint32_t) * rows);
  return hipSuccess;
}

hipError_t launch_compact(const uint64_t* bits, int rows, int, int Tk, int W, int, int run_stride, uint32_t* runs,
                          uint32_t* nruns, uint32_t* live_cnt, uint32_t* heads_ranked, hipStream_t) {
  *heads_ranked = 0;
  uint64_t any = 0;
  for (size_t x = 0; x < (size_t)rows * W; ++x) any |= bits[x];  // reads the whole mask
  for (int r = 0; r < rows; ++r) {                               // one run covering the row: [0, Tk)
    memset(runs + (size_t)r * run_stride, 0, sizeof(uint32_t) * run_stride);
    runs[(size_t)r * run_stride] = (uint32_t)Tk << 16;
    nruns[r] = 1;
    live_cnt[r] = (uint32_t)Tk + (any ? 0u : 0u);
  }
  return hipSuccess;
}

hipError_t launch_clear_tickets(uint32_t* tickets, int stride, hipStream_t) {
  for (int x = 0; x < 8; ++x) tickets[(size_t)x * stride] = 0;
  return hipSuccess;
}

hipError_t launch_prepare_rows(const RowSchedule& p, const uint16_t*, uint16_t* vt, int64_t, int64_t, int64_t, int BH, int,
                               int, int, int Tk, uint32_t* tickets, int ticket_stride, hipStream_t st) {
  if (p.BH > 0) {
    if (*p.heads_ranked != 0) return hipErrorInvalidValue;  // zero between launches
    for (int x = 0; x < p.BH * p.Tq; ++x) p.order[x] = p.live_cnt[x] ? (uint32_t)(x % p.Tq) : 0u;
    for (int u = 0; u < p.chunks; ++u) p.chunk_work[u] = 1;
    if (!before(p.slots + 8 * (size_t)p.per_xcd, p.xcd_rows)) return hipErrorInvalidValue;
    memset(p.slots, 0, sizeof(uint32_t) * 8 * (size_t)p.per_xcd);  // the whole table may be written
    for (int x = 0; x < 8; ++x) p.xcd_rows[x] = 0;
  }
  memset(vt, 0, sizeof(uint16_t) * (size_t)BH * 128 * ((size_t)Tk * 128));
  return tickets ? launch_clear_tickets(tickets, ticket_stride, st) : hipSuccess;
}

hipError_t launch_schedule_rows(const uint64_t* bits, int rows, int, int W, int per_xcd, uint32_t* slots,
                                uint32_t* xcd_rows, hipStream_t) {
  volatile uint64_t sink = bits[0] + bits[(size_t)rows * W - 1];
  (void)sink;
  if (!before(slots + 8 * (size_t)per_xcd, xcd_rows)) return hipErrorInvalidValue;
  memset(slots, 0, sizeof(uint32_t) * 8 * (size_t)per_xcd);
  for (int x = 0; x < 8; ++x) xcd_rows[x] = 0;
  return hipSuccess;
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
  volatile uint32_t sink = 0;
  if (p.scheduled) sink = p.slots[8 * (size_t)p.per_xcd - 1] + p.xcd_rows[7];
  (void)sink;
  if (p.tickets && p.resident == kResident)  // counters start at zero
    for (int x = 0; x < 8; ++x)
      if (!before(p.tickets + x * p.ticket_stride + 1, p.xcd_rows) || p.tickets[x * p.ticket_stride]++ != 0)
        return hipErrorInvalidValue;
  if (p.nseg > 1 && !partials(p, rows * p.nseg, rows)) return hipErrorInvalidValue;
  if (p.piece_units > 0) {
    if (!partials(p, std::max<size_t>(p.piece_units, rows * p.equal_pieces), rows)) return hipErrorInvalidValue;
    for (size_t r = 0; r < rows; ++r)  // arrivals start at zero and are zero again behind the call
      if (p.arrive[r] != 0 || (int)p.live_rows[r] > p.Tk) return hipErrorInvalidValue;
  }
  if (p.cut_rows > 0) {
    const size_t cut = 8 * (size_t)p.cut_rows;
    if (!partials(p, cut * p.cut_pieces, cut)) return hipErrorInvalidValue;
    for (int x = 0; x < 8; ++x)
      for (int r = 0; r < p.cut_rows; ++r) {
        uint32_t* at = p.arrive + x * p.arrive_stride + r;
        // (not the ticket, which the loop above has moved)
        if (!before(at + 1, p.xcd_rows) || *at != 0) return hipErrorInvalidValue;
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
  for (size_t x = 0; x < rows * p.W; ++x) p.bits[x] = p.fresh ? 0 : p.bits[x];
  return hipSuccess;
}

}  // namespace

hipError_t launch_fwd(const FwdParams& p, bool, hipStream_t) {
  const size_t rows = (size_t)p.rows_total;
  if (p.nseg > 0) {
    const hipError_t e = fwd_without_lists(p);
    if (e != hipSuccess) return e;
  } else {
    // the first and last element of everything the kernel reads or writes besides q, k, v, out
    volatile uint32_t sink = p.runs[0] + p.runs[rows * p.run_stride - 1] + p.nruns[rows - 1] + p.live_cnt[rows - 1] +
                             p.slots[8 * (size_t)p.per_xcd - 1] + p.xcd_rows[7] +
                             p.vt[(size_t)(rows / p.Tq) * 128 * ((size_t)p.Tk * 128) - 1];
    (void)sink;
    p.bits[0] |= 0;
    p.bits[rows * p.W - 1] |= 0;
    if (p.build_next) {  // the epilogue rewrites the lists in full
      memset(p.runs, 0, sizeof(uint32_t) * rows * p.run_stride);
      for (size_t r = 0; r < rows; ++r) {
        p.runs[r * p.run_stride] = (uint32_t)p.Tk << 16;
        p.nruns[r] = 1;
        p.live_cnt[r] = (uint32_t)p.Tk;
      }
    }
  }
  *p.stat_skipped_in += 0;
  *p.stat_newly += 0;
  *p.stat_runs += (unsigned long long)rows;
  return hipSuccess;
}

}  // namespace la
