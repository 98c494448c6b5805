// Host side of the C ABI declared in include/lite_attn.h: handles, contexts, launches (argument checks and buffer
// layouts are in lite_attn_host.cpp).
#include "lite_attn.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <new>

#include "lite_attn_kernels.h"

// Device memory that every call rewrites before reading it (nothing in it outlives a call): V^T or partial results.  A
// handle either owns one or borrows its context's; empty if no layer needs any.
struct la_scratch {
  void* base = nullptr;
  size_t bytes = 0;
};

struct lite_attn_ctx {
  la_scratch scratch;
  hipStream_t stream = nullptr;
  int device = 0;
  int handles = 0;  // live handles attached to this context
};

struct lite_attn_mask {
  lite_attn_desc_t desc;
  la::Geometry geo;
  la::ListLayout ll;
  uint64_t* d_bits;
  char* d_lists;      // Skip-Lists and row ranking (layout ll); kept between calls
  int table_calls;    // calls that the row schedule has served; 0: there is none that can serve another
  float loosest;        // largest threshold of the trajectory's calls so far (-inf: none has marked)
  float table_loosest;  // what it was when the row schedule was made
  unsigned long long capture;  // the capture that the last call was recorded in; 0: it ran
  bool recorded;               // a call has been recorded: it may run again whenever its graph is replayed
  bool lists_valid;   // the lists describe the mask as it stands (left by the previous call's epilogue, or an import)
  unsigned long long* d_stats;  // [max_steps][3]: skipped on entry, newly marked, Skip-List runs
  uint32_t* d_newly;            // few rows, behind them: [kFewRows] tiles that step 0 marked, per row (part of step
                                //   0's newly marked)
  uint32_t* d_arrive;           // behind it, [kFewRows] arrivals of rows cut into pieces, zero between calls; behind them
                                //   [2][kFewRows] live tiles of the rows (live_rows())
  bool empty;                   // nothing can have marked a tile since step 0
  la_scratch own;               // used when ctx == nullptr
  lite_attn_ctx* ctx;           // shared scratch + stream, or nullptr
  hipStream_t stream;           // used when ctx == nullptr
  int next_step;
  bool profile;
  hipEvent_t* events;  // [max_steps][3] once profiling was enabled: before the pre-passes, between, after attention
  bool* timed;         // [max_steps]
};

namespace {
thread_local int g_last_hip = 0;
}

namespace la {

int hip_fail(hipError_t e) {
  g_last_hip = (int)e;
  return e == hipErrorOutOfMemory ? LITE_ATTN_ENOMEM : LITE_ATTN_EHIP;
}

hipError_t launch_call(const lite_attn_desc_t& d, const Geometry& g, const ListLayout& ll, char* lists, char* scratch,
                       const CallArgs& a, hipStream_t stream, hipEvent_t mid) {
  uint32_t* runs = reinterpret_cast<uint32_t*>(lists + ll.runs);
  uint32_t* nruns = reinterpret_cast<uint32_t*>(lists + ll.nruns);
  uint32_t* live_cnt = reinterpret_cast<uint32_t*>(lists + ll.live_cnt);
  uint32_t* slots = reinterpret_cast<uint32_t*>(lists + ll.slots);
  uint32_t* xcd_rows = reinterpret_cast<uint32_t*>(lists + ll.xcd_rows);
  uint32_t* heads_ranked = reinterpret_cast<uint32_t*>(lists + ll.heads_ranked);
  uint32_t* own_tickets = reinterpret_cast<uint32_t*>(lists + ll.tickets);
  uint16_t* vt = reinterpret_cast<uint16_t*>(scratch);
  const int diagonal_first = (d.flags & LITE_ATTN_ORDER_DIAGONAL_FIRST) ? 1 : 0;
  const bool few = g.nseg > 0;
  hipError_t e = hipSuccess;
  // a table of rows comes with its ticket counters cleared; calls without one have theirs apart, as later calls, recorded
  // ones above all, may go by a table that is in place
  const bool table = !few || (g.rows > kFewRows && g.rows <= kSchedRows && !a.empty);
  const bool tickets = g.rows > kFewRows, draws = tickets && (!few || g.Tk >= kDrawTiles);
  if (!few && a.fresh) {
    e = launch_clear(a.bits, (size_t)g.rows * g.W, a.stats_all, a.stat_words, stream);
  } else if (tickets && !table && (draws || a.fresh)) {  // (the mask is overwritten; few rows: the kernel clears)
    e = launch_clear(reinterpret_cast<uint64_t*>(own_tickets), draws ? 8 * (kTicketWords + kArrivals) / 2 : 0, a.stats_all,
                     a.fresh ? a.stat_words : 0, stream);
  }
  if (e != hipSuccess) return e;
  if (!few) {
    uint32_t* order = reinterpret_cast<uint32_t*>(lists + ll.order);
    uint32_t* chunk_work = reinterpret_cast<uint32_t*>(lists + ll.chunk_work);
    if (!a.lists_ready) {
      e = launch_compact(a.bits, (int)g.rows, g.Tq, g.Tk, g.W, diagonal_first, g.run_stride, runs, nruns, live_cnt,
                         heads_ranked, stream);
      if (e != hipSuccess) return e;
    }
    const RowSchedule sched = {live_cnt, order, chunk_work, slots, xcd_rows, heads_ranked, g.Tq, g.Tk, g.BH, g.chunks,
                               g.per_xcd};
    e = launch_prepare_rows(sched, static_cast<const uint16_t*>(a.v), vt, d.stride_b, d.stride_h, d.stride_n, d.heads,
                            d.seqlen, stream);
    if (e != hipSuccess) return e;
  }
  FwdParams p;
  p.q = static_cast<const uint16_t*>(a.q);
  p.k = static_cast<const uint16_t*>(a.k);
  p.vt = vt;
  p.out = static_cast<uint16_t*>(a.out);
  p.stride_b = d.stride_b; p.stride_h = d.stride_h; p.stride_n = d.stride_n;
  p.H = d.heads; p.N = d.seqlen; p.Tq = g.Tq; p.Tk = g.Tk; p.W = g.W;
  p.runs = runs; p.run_stride = g.run_stride; p.nruns = nruns; p.live_cnt = live_cnt;
  p.bits = a.bits;
  p.stat_skipped_in = a.stats3;
  p.stat_newly = a.stats3 ? a.stats3 + 1 : nullptr;
  p.stat_runs = a.stats3 ? a.stats3 + 2 : nullptr;
  p.thr = a.threshold;
  p.scale = 1.0f / std::sqrt((float)d.head_dim);
  p.protect_start = d.protect_start; p.protect_len = d.protect_len;
  p.rows_total = (int)g.rows;
  p.slots = slots; p.per_xcd = g.per_xcd; p.xcd_rows = xcd_rows;
  p.tickets = !tickets ? nullptr : table ? slots + g.per_xcd - 1 : own_tickets;
  p.ticket_stride = table ? g.per_xcd : kTicketWords;
  p.resident = draws ? kResident : kNoDraws;
  p.table_calls = a.table_calls;
  p.build_next = a.build_next ? 1 : 0;
  p.diagonal_first = diagonal_first;
  if (few) {
    p.nseg = g.nseg;
    p.pair = g.pair;
    p.fresh = a.fresh ? 1 : 0;
    p.v = static_cast<const uint16_t*>(a.v);
    // (a call that marks nothing is one of dense attention in all likelihood: its rows are alike)
    if (g.pieces > 0 && g.rows <= kFewRows && a.threshold > -INFINITY) {
      p.pair = g.pieces == kPairWorkgroups ? 1 : 0;
      p.nseg = equal_pieces(g);
      // Pieces by the rows' live tiles, or, where these turn out to be all, the same number of each.  Where they are
      // known to be all, segments and merge pass unless the pieces run in one round and have few row maxima to walk:
      // us, step 0, merge pass -> last piece, 80 x 16 27.4 -> 25.1, 120 x 20 36.4 -> 33.5, 105 x 35 46.8 -> 46.1; 128 x
      // 64 80.8 -> 81.0, 99 x 99 102.1 -> 103.0; in two rounds 344 x 86 258 -> 295, as the second's workgroups then
      // meet in pairs on the CUs that end first.
      if (!a.empty || (p.nseg > 1 && g.rows * p.nseg <= g.pieces && g.Tk < 64)) {
        p.alike = a.empty ? 1 : 0;
        p.equal_pieces = p.nseg;
        p.nseg = 1;
        p.piece_units = g.pieces;
        p.arrive = a.arrive;
        p.live_rows = a.live_rows;
        if (!p.arrive) {  // (where the table and the lists would be)
          uint32_t* live = reinterpret_cast<uint32_t*>(lists + ll.live_cnt);
          p.arrive = slots;
          p.live_rows = live;
          e = launch_count_rows(a.bits, (int)g.rows, g.Tk, g.W, live, slots, stream);
          if (e != hipSuccess) return e;
        }
      }
    }
    if (cut_rows(g) > 0) {
      p.cut_rows = cut_rows(g);
      p.cut_pieces = cut_pieces(g);
      p.arrive = table ? slots + g.per_xcd - 1 - kArrivals : own_tickets + 8 * kTicketWords;
      p.arrive_stride = table ? g.per_xcd : kArrivals;
      p.marked = table ? slots + g.per_xcd - kTableTail + 1 : nullptr;
    }
    if (p.nseg > 1 || p.piece_units > 0 || p.cut_rows > 0) {
      const ScratchLayout sl = scratch_layout(g, p.nseg);
      p.seg_o = reinterpret_cast<float*>(scratch + sl.seg_o);
      p.seg_stat = reinterpret_cast<float*>(scratch + sl.seg_stat);
      p.seg_mloc = reinterpret_cast<float*>(scratch + sl.seg_mloc);
    }
    p.stats_all = a.stats_all;
    p.newly_rows = a.newly_rows;
    p.live_next = a.live_next;
    p.stat_words = (int64_t)a.stat_words;
    if (a.fresh && a.newly_rows && p.stat_words > (int64_t)kClearWords * 256 * p.rows_total * p.nseg * p.equal_pieces) {
      e = launch_clear(a.bits, 0, a.stats_all, a.stat_words, stream);
      if (e != hipSuccess) return e;
      p.stat_words = 3;  // (step 0's, which do not start at zero)
    }
    // nothing to schedule where all workgroups start together or all rows are equally long; beyond kSchedRows rows the
    // kernel deals chunks of them in turn
    if (table) {
      p.scheduled = 1;
      if (a.table_calls == 0)
        e = launch_schedule_rows(a.bits, (int)g.rows, g.Tk, g.W, g.per_xcd, slots, xcd_rows, stream);
      else if (draws)
        e = launch_clear_tickets(p.tickets, p.ticket_stride, stream);
      if (e != hipSuccess) return e;
    }
  }
  p.parts = few ? p.nseg * p.equal_pieces : 1;
  p.per_Tq = reciprocal(g.Tq);
  p.per_H = reciprocal(d.heads);
  p.per_parts = reciprocal(p.parts);
  if (mid) {
    e = hipEventRecord(mid, stream);
    if (e != hipSuccess) return e;
  }
  return launch_fwd(p, (d.flags & LITE_ATTN_PV_SKIP_IMMEDIATE) != 0, stream);
}

}  // namespace la

namespace {

using la::hip_fail;

#define LA_HIP(expr)                           \
  do {                                         \
    hipError_t e_ = (expr);                    \
    if (e_ != hipSuccess) return hip_fail(e_); \
  } while (0)

hipStream_t stream_of(const lite_attn_mask* m) { return m->ctx ? m->ctx->stream : m->stream; }
char* scratch_of(const lite_attn_mask* m) { return static_cast<char*>(m->ctx ? m->ctx->scratch.base : m->own.base); }
// Layers of few rows that may be cut into pieces: the rows' live tiles at the start of `step`, left by the call before
// or by an import (two sets in turn, as a call reads one while it leaves the other).
uint32_t* live_rows(const lite_attn_mask* m, int step) {
  if (m->geo.pieces == 0 || m->geo.rows > la::kFewRows) return nullptr;
  return m->d_arrive + (1 + (step & 1)) * la::kFewRows;
}

// The capture under way on a stream, 0 if there is none (the null stream cannot be captured, and may not be asked while
// another stream is).  False if the runtime does not tell: no reason to refuse a call.
bool capture_on(hipStream_t stream, unsigned long long* capture) {
  *capture = 0;
  if (!stream || stream == hipStreamLegacy) return true;
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  if (hipStreamGetCaptureInfo(stream, &status, &id) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (status != hipStreamCaptureStatusNone) *capture = id + 1;
  return true;
}

// The Skip-Lists of the mask as it stands.  A handle of a layer that has them keeps them in line with its mask from the first,
// as a recorded later call reads them whatever has happened since it was recorded.
hipError_t make_lists(const lite_attn_mask* m, hipStream_t stream) {
  const la::Geometry& g = m->geo;
  const la::ListLayout& l = m->ll;
  auto at = [&](size_t offset) { return reinterpret_cast<uint32_t*>(m->d_lists + offset); };
  return la::launch_compact(m->d_bits, (int)g.rows, g.Tq, g.Tk, g.W, m->desc.flags & LITE_ATTN_ORDER_DIAGONAL_FIRST,
                            g.run_stride, at(l.runs), at(l.nruns), at(l.live_cnt), at(l.heads_ranked), stream);
}

int grow(la_scratch* s, size_t bytes) {
  if (bytes <= s->bytes) return LITE_ATTN_OK;
  if (s->base) LA_HIP(hipFree(s->base));
  s->base = nullptr;
  s->bytes = 0;
  LA_HIP(hipMalloc(&s->base, bytes));
  s->bytes = bytes;
  return LITE_ATTN_OK;
}

int init_common(const lite_attn_desc_t* desc, lite_attn_ctx* ctx, lite_attn_mask_t** out) {
  if (!out) return LITE_ATTN_EINVAL;
  int rc = la::check_desc(desc);
  if (rc != LITE_ATTN_OK) return rc;
  lite_attn_mask* m = new (std::nothrow) lite_attn_mask();
  if (!m) return LITE_ATTN_ENOMEM;
  m->desc = *desc;
  m->geo = la::geometry(*desc);
  m->ll = la::list_layout(m->geo);
  m->d_lists = nullptr;
  m->lists_valid = false;
  m->table_calls = 0;
  m->loosest = m->table_loosest = -INFINITY;
  m->capture = 0;
  m->recorded = false;
  m->ctx = nullptr;
  m->stream = nullptr;
  m->next_step = 0;
  m->profile = false;
  m->events = nullptr;
  m->timed = nullptr;
  m->d_bits = nullptr;
  m->d_stats = nullptr;
  m->d_newly = nullptr;
  m->d_arrive = nullptr;
  m->empty = false;
  const size_t words = (size_t)m->geo.rows * m->geo.W, nstats = 3 * (size_t)desc->max_steps;
  const size_t counters = m->geo.rows <= la::kFewRows ? 4 * la::kFewRows * sizeof(uint32_t) / sizeof(unsigned long long) : 0;
  const size_t need = la::scratch_layout(m->geo).total;
  hipStream_t st = ctx ? ctx->stream : nullptr;
  rc = LITE_ATTN_OK;
  if (ctx) {
    // every call made so far through this context has to finish before its scratch may move
    hipError_t e = need > ctx->scratch.bytes ? hipStreamSynchronize(ctx->stream) : hipSuccess;
    rc = e != hipSuccess ? hip_fail(e) : grow(&ctx->scratch, need);
  } else {
    rc = grow(&m->own, need);
  }
  if (rc == LITE_ATTN_OK) {
    hipError_t e = hipMalloc(&m->d_bits, sizeof(uint64_t) * words);
    if (e == hipSuccess) e = hipMalloc(&m->d_stats, sizeof(unsigned long long) * (nstats + counters));
    if (e == hipSuccess) e = hipMalloc(&m->d_lists, m->ll.total);
    if (e == hipSuccess) e = la::prepare_fwd();
    if (e == hipSuccess) e = la::launch_clear(m->d_bits, words, m->d_stats, nstats + counters, st);
    if (e == hipSuccess && counters) {
      m->d_newly = reinterpret_cast<uint32_t*>(m->d_stats + nstats);
      m->d_arrive = m->d_newly + la::kFewRows;
    }
    if (e == hipSuccess && m->geo.nseg == 0) e = make_lists(m, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) rc = hip_fail(e);
  }
  if (rc != LITE_ATTN_OK) {
    lite_attn_free_mask(m);
    return rc;
  }
  if (ctx) {
    m->ctx = ctx;
    ++ctx->handles;
  }
  *out = m;
  return LITE_ATTN_OK;
}

}  // namespace

extern "C" {

int lite_attn_init_mask(const lite_attn_desc_t* desc, lite_attn_mask_t** out) { return init_common(desc, nullptr, out); }

int lite_attn_ctx_create(lite_attn_ctx_t** out) {
  if (!out) return LITE_ATTN_EINVAL;
  lite_attn_ctx* c = new (std::nothrow) lite_attn_ctx();
  if (!c) return LITE_ATTN_ENOMEM;
  hipError_t e = hipGetDevice(&c->device);
  if (e != hipSuccess) {
    delete c;
    return hip_fail(e);
  }
  *out = c;
  return LITE_ATTN_OK;
}

int lite_attn_ctx_set_stream(lite_attn_ctx_t* ctx, void* hip_stream) {
  if (!ctx) return LITE_ATTN_EINVAL;
  LA_HIP(hipStreamSynchronize(ctx->stream));  // work already queued keeps its order with what follows
  ctx->stream = reinterpret_cast<hipStream_t>(hip_stream);
  return LITE_ATTN_OK;
}

int lite_attn_init_mask_shared(const lite_attn_desc_t* desc, lite_attn_ctx_t* ctx, lite_attn_mask_t** out) {
  if (!ctx) return LITE_ATTN_EINVAL;
  return init_common(desc, ctx, out);
}

int lite_attn_ctx_free(lite_attn_ctx_t* ctx) {
  if (!ctx) return LITE_ATTN_OK;
  if (ctx->handles != 0) return LITE_ATTN_ESHARED;
  if (ctx->scratch.base) (void)hipFree(ctx->scratch.base);
  delete ctx;
  return LITE_ATTN_OK;
}

int lite_attn_set_stream(lite_attn_mask_t* m, void* hip_stream) {
  if (!m) return LITE_ATTN_EINVAL;
  if (m->ctx)  // the scratch is only safe while every handle of the context runs on the context's one stream
    return reinterpret_cast<hipStream_t>(hip_stream) == m->ctx->stream ? LITE_ATTN_OK : LITE_ATTN_ESHARED;
  LA_HIP(hipStreamSynchronize(m->stream));  // work already queued keeps its order with what follows
  m->stream = reinterpret_cast<hipStream_t>(hip_stream);
  return LITE_ATTN_OK;
}

int lite_attn_fwd(const void* q, const void* k, const void* v, void* out, lite_attn_mask_t* m, float threshold,
                  int step) {
  if (!m) return LITE_ATTN_EINVAL;
  int rc = la::check_call(q, k, v, out, threshold);
  if (rc != LITE_ATTN_OK) return rc;
  if (step < 0 || step >= m->desc.max_steps) return LITE_ATTN_ESTEP;
  if (step != 0 && step != m->next_step) return LITE_ATTN_ESTEP;
  const lite_attn_desc_t& d = m->desc;
  hipStream_t stream = stream_of(m);
  hipEvent_t* ev = (m->profile && m->events) ? m->events + 3 * (size_t)step : nullptr;
  if (m->timed) m->timed[step] = ev != nullptr;
  if (ev) LA_HIP(hipEventRecord(ev[0], stream));
  // Lists left by the previous call's epilogue, or an import, are used: not at step 0 (the mask was just cleared).  This call's
  // epilogue then leaves the lists of the next call.
  const bool ready = m->lists_valid && step != 0;
  m->lists_valid = false;
  // A recorded call runs when its graph is replayed, of which the host hears nothing: what it knows of the device's state (an
  // empty mask, a row schedule that fits) holds among the calls of one capture, and among eager ones while no call has been
  // recorded.  Elsewhere a call finds out for itself, with the same bits.
  unsigned long long capture;
  const bool told = capture_on(stream, &capture);
  const bool known = told && capture == m->capture && (capture != 0 || !m->recorded);
  m->capture = capture;
  m->recorded = m->recorded || !told || capture != 0;
  la::CallArgs a;
  a.q = q; a.k = k; a.v = v; a.out = out;
  a.threshold = threshold;
  a.bits = m->d_bits;
  a.stats3 = m->d_stats + 3 * (size_t)step;
  a.fresh = step == 0;
  a.stats_all = m->d_stats;
  a.stat_words = 3 * (size_t)d.max_steps;
  a.newly_rows = m->d_newly;
  a.arrive = m->d_arrive;
  a.live_rows = live_rows(m, step);
  a.live_next = live_rows(m, step + 1);
  a.empty = step == 0 || (known && m->empty);
  a.lists_ready = ready;
  a.build_next = true;
  // The row schedule serves up to kTableCalls calls of a trajectory, as long as no call has marked with a looser threshold
  // than the mask that it was made for has seen: what a threshold marks, it marks nearly all at once.
  if (step == 0) m->loosest = -INFINITY;
  const bool keeps = la::keeps_table(m->geo) && !a.empty;
  const bool ready_table = keeps && known && m->table_calls < la::kTableCalls && m->table_loosest == m->loosest;
  a.table_calls = ready_table ? m->table_calls : 0;
  const int served = keeps ? a.table_calls + 1 : 0;
  m->table_calls = 0;
  LA_HIP(la::launch_call(d, m->geo, m->ll, m->d_lists, scratch_of(m), a, stream, ev ? ev[1] : nullptr));
  m->lists_valid = m->geo.nseg == 0;  // (calls with few or short rows keep no lists)
  m->table_calls = served;
  m->table_loosest = m->loosest;
  m->loosest = std::fmax(m->loosest, threshold);
  m->empty = a.empty && !(threshold > -INFINITY);
  if (ev) LA_HIP(hipEventRecord(ev[2], stream));
  m->next_step = step + 1;
  return LITE_ATTN_OK;
}

int lite_attn_skip_stats(lite_attn_mask_t* m, int step, lite_attn_stats_t* host_out) {
  if (!m || !host_out) return LITE_ATTN_EINVAL;
  if (step < 0 || step >= m->next_step || step >= m->desc.max_steps) return LITE_ATTN_ESTEP;
  unsigned long long raw[3];
  LA_HIP(hipMemcpyAsync(raw, m->d_stats + 3 * (size_t)step, sizeof raw, hipMemcpyDeviceToHost, stream_of(m)));
  uint32_t newly[la::kFewRows] = {};
  if (step == 0 && m->d_newly)
    LA_HIP(hipMemcpyAsync(newly, m->d_newly, sizeof newly, hipMemcpyDeviceToHost, stream_of(m)));
  LA_HIP(hipStreamSynchronize(stream_of(m)));
  for (const uint32_t n : newly) raw[1] += n;
  host_out->step = step;
  host_out->tiles_total = (uint64_t)m->geo.rows * (uint64_t)m->geo.Tk;
  host_out->tiles_skipped_in = raw[0];
  host_out->tiles_newly_marked = raw[1];
  host_out->live_list_bytes = raw[2] * sizeof(uint32_t);
  return LITE_ATTN_OK;
}

int lite_attn_profile(lite_attn_mask_t* m, int enable) {
  if (!m) return LITE_ATTN_EINVAL;
  if (enable && !m->events) {
    const size_t n = 3 * (size_t)m->desc.max_steps;
    hipEvent_t* ev = new (std::nothrow) hipEvent_t[n];
    bool* timed = new (std::nothrow) bool[m->desc.max_steps]();
    if (!ev || !timed) {
      delete[] ev;
      delete[] timed;
      return LITE_ATTN_ENOMEM;
    }
    for (size_t x = 0; x < n; ++x) {
      hipError_t e = hipEventCreate(&ev[x]);
      if (e != hipSuccess) {
        for (size_t y = 0; y < x; ++y) (void)hipEventDestroy(ev[y]);
        delete[] ev;
        delete[] timed;
        return hip_fail(e);
      }
    }
    m->events = ev;
    m->timed = timed;
  }
  m->profile = enable != 0;
  return LITE_ATTN_OK;
}

int lite_attn_kernel_times(lite_attn_mask_t* m, int step, float* host_prep_ms, float* host_fwd_ms) {
  if (!m || !host_prep_ms || !host_fwd_ms) return LITE_ATTN_EINVAL;
  if (step < 0 || step >= m->desc.max_steps || !m->events || !m->timed[step]) return LITE_ATTN_ESTEP;
  hipEvent_t* ev = m->events + 3 * (size_t)step;
  LA_HIP(hipEventSynchronize(ev[2]));
  LA_HIP(hipEventElapsedTime(host_prep_ms, ev[0], ev[1]));
  LA_HIP(hipEventElapsedTime(host_fwd_ms, ev[1], ev[2]));
  return LITE_ATTN_OK;
}

size_t lite_attn_mask_words(const lite_attn_mask_t* m) { return m ? (size_t)m->geo.rows * m->geo.W : 0; }

int lite_attn_mask_export(lite_attn_mask_t* m, uint64_t* host_bits, size_t words) {
  if (!m || !host_bits || words != lite_attn_mask_words(m)) return LITE_ATTN_EINVAL;
  LA_HIP(hipMemcpyAsync(host_bits, m->d_bits, words * sizeof(uint64_t), hipMemcpyDeviceToHost, stream_of(m)));
  LA_HIP(hipStreamSynchronize(stream_of(m)));
  return LITE_ATTN_OK;
}

int lite_attn_mask_import(lite_attn_mask_t* m, const uint64_t* host_bits, size_t words, int next_step) {
  if (!m || !host_bits || words != lite_attn_mask_words(m)) return LITE_ATTN_EINVAL;
  if (next_step < 0 || next_step >= m->desc.max_steps) return LITE_ATTN_ESTEP;
  LA_HIP(hipMemcpyAsync(m->d_bits, host_bits, words * sizeof(uint64_t), hipMemcpyHostToDevice, stream_of(m)));
  if (uint32_t* live = live_rows(m, next_step))
    LA_HIP(la::launch_count_rows(m->d_bits, (int)m->geo.rows, m->geo.Tk, m->geo.W, live, nullptr, stream_of(m)));
  if (m->geo.nseg == 0) LA_HIP(make_lists(m, stream_of(m)));
  LA_HIP(hipStreamSynchronize(stream_of(m)));
  m->next_step = next_step;
  m->empty = false;
  m->table_calls = 0;
  m->lists_valid = m->geo.nseg == 0;
  return LITE_ATTN_OK;
}

int lite_attn_skipruns_export(lite_attn_mask_t* m, uint32_t* host_runs, uint32_t* host_nruns) {
  if (!m || !host_runs || !host_nruns) return LITE_ATTN_EINVAL;
  const la::Geometry& g = m->geo;
  uint32_t* runs = reinterpret_cast<uint32_t*>(m->d_lists + m->ll.runs);
  uint32_t* nruns = reinterpret_cast<uint32_t*>(m->d_lists + m->ll.nruns);
  hipStream_t stream = stream_of(m);
  // (if the lists were already in place -- left by the last call's epilogue -- this writes the same values again)
  LA_HIP(make_lists(m, stream));
  LA_HIP(hipMemcpyAsync(host_runs, runs, sizeof(uint32_t) * (size_t)g.rows * g.run_stride, hipMemcpyDeviceToHost,
                        stream));
  LA_HIP(hipMemcpyAsync(host_nruns, nruns, sizeof(uint32_t) * (size_t)g.rows, hipMemcpyDeviceToHost, stream));
  LA_HIP(hipStreamSynchronize(stream));
  return LITE_ATTN_OK;
}

size_t lite_attn_skipruns_stride(const lite_attn_mask_t* m) { return m ? (size_t)m->geo.run_stride : 0; }

int lite_attn_skiplist_export(lite_attn_mask_t* m, uint16_t* host_live_idx, uint32_t* host_live_cnt) {
  if (!m || !host_live_idx || !host_live_cnt) return LITE_ATTN_EINVAL;
  const la::Geometry& g = m->geo;
  uint32_t* runs = new (std::nothrow) uint32_t[(size_t)g.rows * g.run_stride];
  uint32_t* nruns = new (std::nothrow) uint32_t[(size_t)g.rows];
  int rc = (runs && nruns) ? lite_attn_skipruns_export(m, runs, nruns) : LITE_ATTN_ENOMEM;
  if (rc == LITE_ATTN_OK) {
    for (int64_t row = 0; row < g.rows; ++row) {  // expand the runs into the packed index list
      uint32_t n = 0;
      for (uint32_t x = 0; x < nruns[row]; ++x) {
        const uint32_t e = runs[row * g.run_stride + x];
        for (uint32_t j = e & 0xffffu; j < (e >> 16); ++j) host_live_idx[row * g.Tk + n++] = (uint16_t)j;
      }
      host_live_cnt[row] = n;
    }
  }
  delete[] runs;
  delete[] nruns;
  return rc;
}

void lite_attn_free_mask(lite_attn_mask_t* m) {
  if (!m) return;
  if (m->ctx) {
    // the shared scratch stays with the context; calls of this handle still in flight only touch the scratch and
    // the buffers freed below, and hipFree waits for the device
    --m->ctx->handles;
  }
  if (m->d_bits) (void)hipFree(m->d_bits);
  if (m->d_stats) (void)hipFree(m->d_stats);
  if (m->d_lists) (void)hipFree(m->d_lists);
  if (m->own.base) (void)hipFree(m->own.base);
  if (m->events) {
    for (size_t x = 0; x < 3 * (size_t)m->desc.max_steps; ++x) (void)hipEventDestroy(m->events[x]);
    delete[] m->events;
  }
  delete[] m->timed;
  delete m;
}

const char* lite_attn_strerror(int code) {
  switch (code) {
    case LITE_ATTN_OK: return "ok";
    case LITE_ATTN_EINVAL: return "invalid argument";
    case LITE_ATTN_ESTEP: return "step out of sequence";
    case LITE_ATTN_EUNSUPPORTED: return "unsupported shape (head_dim and tiles must be 128)";
    case LITE_ATTN_ENOMEM: return "out of memory";
    case LITE_ATTN_EHIP: return "HIP runtime error";
    case LITE_ATTN_ESHARED:
      return "not allowed while scratch is shared (a handle of a context runs on the context's stream; a context "
             "with live handles cannot be freed)";
    case LITE_ATTN_ESCRATCH: return "the shape needs more scratch than the static device array holds";
    default: return "unknown error";
  }
}

int lite_attn_last_hip_error(void) { return g_last_hip; }

}  // extern "C"
