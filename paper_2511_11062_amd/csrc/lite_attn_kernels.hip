// gfx950 (CDNA4) kernels of the LiteAttention forward path.
//
//   clear_state_kernel   : zero the Skip-Mask and the statistics (step 0)
//   compact_skiplist     : Skip-Mask row -> run-length list of its live K/V tiles, (start,end) per run
//                          (Implementation, "Producer and Skip-List Optimization"); only at the start of a trajectory
//                          or after a mask import: the fused kernel's epilogue builds the next call's Skip-Lists
//   prepare_rows_kernel  : per head, Q-tile rows ranked by Skip-List length and the ranked rows dealt to the XCDs (the
//                          launch order of the fused kernel), beside V -> V^T scratch, so that the PV operand is read from
//                          LDS like the QK operand
//   schedule_rows_kernel : the row schedule of layers with short rows, from the mask itself
//   merge_segments_kernel: partial results of rows that were cut into segments -> O, mask bits, statistics
//   lite_attn_fwd_kernel : fused tiled forward over the live tiles with the skip predicate
//                          (Algorithm 2; eq. sparge_cond; tile recurrences of the Preliminaries)
//
// Fused kernel, one workgroup (4 wave64) = one Q tile = one Skip-Mask row:
//   * wave w owns Q rows [32w, 32w+32); lane l owns Q row (l & 31) of them.
//   * it works on S^T = K Q^T with v_mfma_f32_32x32x16_bf16: K rows are the A operand (LDS), Q rows the B
//     operand (registers, loaded once), so the 16 accumulator values a lane holds per 32x32 block all belong
//     to ONE Q row: row max / row sum are in-lane reductions plus one v_permlane32_swap, and exp(S^T) in
//     accumulator layout IS the B operand of O^T = V^T P^T -- P never moves between lanes.
//   * a 128-column mask tile is streamed as two 64-column stages.  K and V stages go global -> LDS with
//     buffer_load ... lds (no registers, rows past the end of the sequence arrive as zeros through the buffer
//     descriptor's range check); both are stored unpadded with an XOR swizzle applied on the global-address
//     side.  V is transposed once per call into a scratch (prepare_rows_kernel), so that K and V^T fragments are
//     both plain 16-byte LDS reads.
//   * software pipeline: in stage s the matrix cores run S(s+1) = K(s+1) Q^T and O += V(s-1) P(s-1) while the
//     vector ALU runs the online softmax of stage s; LDS holds two K and two V stages (64 KB), one barrier per
//     stage, two workgroups per CU.
//   * the predicate of a tile is reduced per wave with a ballot; the four per-wave results meet through LDS
//     at the barrier that ends the tile and one lane ORs the bit into the global mask row.
//   * IMM variant (Algorithm 2 taken literally: a tile that fires contributes nothing in the step that marks it):
//     O += V(s-2) P(s-2) runs two stages behind instead of one, so that the verdict on a tile is known before the
//     first of its two PV products is issued; a fired tile's PV MFMAs and row sums are then dropped.
//
// Calls with few rows (at most kFewRows = 512, which all fit the chip at once) or short rows (at most kShortTiles = 192
// tiles, any number of them up to kMaxListless) take the template argument FEW of the fused kernel.  The former are
// bound by launches and by latency, not by the matrix cores: the tiny layer's step was 36 us of attention on 32 of 256
// CUs behind four to six launches of 4 us each; for the latter the passes before the kernel cost more than they save.
// They run in one or two launches:
//   * no lists and no ranking: a workgroup finds its live tiles from the mask row itself (LiveWalk); more than kFewRows rows
//     are scheduled from the mask in one launch (schedule_rows_kernel; not at step 0 and not beyond kSchedRows rows);
//   * no V^T: the V fragments come from V as it lies in memory through transposing LDS reads (ds_read_b64_tr_b16), 16 LDS
//     instructions more per stage, the same LDS cycles (no bank conflicts): 1.8 % of the kernel's time on the 12-head
//     N = 32760 dense step, against a launch and a pass over V;
//   * with few rows a workgroup may be a PAIR of groups of four waves, each with its own stage buffers and one
//     64-column half of every tile (a CU with one wave per SIMD issues too slowly to keep the matrix cores busy); the
//     groups' results meet in LDS at the end, their row maxima once per tile, for the predicate;
//   * with few rows a row may be cut into segments, one workgroup each (the rule and its measurements: share_chip() in
//     lite_attn_host.cpp); merge_segments_kernel adds up the partial results.  The predicate stays exact: the
//     segments record every tile's row maxima, and the merge pass judges them against the running maximum carried
//     over the segments, the value a single pass would have had;
//   * under a mask rows may be cut by their live tiles, into pieces of about equal length (pick_piece), merged by the
//     workgroup that finishes last.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <stdint.h>

#include <utility>

#include "lite_attn_kernels.h"

namespace la {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

#define LA_LDS __attribute__((address_space(3)))

// f(integral_constant<int, 0>), f(integral_constant<int, 1>), ... : a loop whose index is a constant expression
template <int... Ks, class F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, Ks...>, F&& f) {
  (f(std::integral_constant<int, Ks>{}), ...);
}

// Stores past the XCD's L2 (scope bit sc1, the agent scope), for what the next launch reads: a line left in the L2 is
// written back at the end of the kernel, and that launch waits for it (5 us behind a call that leaves 16 MB of partial
// results, 2 us behind one without).
constexpr int kStoreThrough = 16;  // cache policy of a buffer store
template <class T>
__device__ __forceinline__ void store_through(T* at, T x) {
  __hip_atomic_store(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kTile = 128;        // Skip-Mask tile: 128 Q rows x 128 K/V columns
constexpr int kSub = 64;          // K/V columns per pipeline stage
constexpr int kStageBytes = kSub * 256;  // one K or V stage: 64 rows x 128 bf16, unpadded
constexpr int kKOff = 0;                 // K stage p at kKOff + p * kStageBytes
constexpr int kVOff = 2 * kStageBytes;   // V stage p at kVOff + p * kStageBytes
constexpr int kFlagsOff = 4 * kStageBytes;  // 8 ints [tile parity][wave] + 64 dummy ints
constexpr int kFiredOff = kFlagsOff + 8 * 4 + 64 * 4;  // W uint64: mask bits this workgroup set during the call
constexpr int kMaxMaskWords = 256;                     // ceil(16383 / 64)
constexpr int kLdsBytes = kFiredOff + 8 * kMaxMaskWords;
// PAIR: two sets of stage buffers, then the flags, then group 1's row maxima [tile parity][128]
constexpr int kPairFlagsOff = 8 * kStageBytes;
constexpr int kPairXchOff = kPairFlagsOff + 8 * 4 + 64 * 4;
constexpr int kPairLdsBytes = kPairXchOff + 2 * kTile * 4;
constexpr int kORow = 272;        // bytes per O row in the epilogue staging (reuses the stage buffers)

constexpr int kRowsPerWave = 8;  // Q-tile rows compacted by one wave of compact_skiplist

// Brings the kernel's arguments into the scalar cache, all lines at once: they come from host memory, and left to the
// places of their first use a workgroup would wait for one line after the other.
__device__ __forceinline__ void touch_arguments(size_t bytes) {
  typedef const __attribute__((address_space(4))) uint32_t* words;
  const words a = (words)__builtin_amdgcn_kernarg_segment_ptr();
  const int last = (int)bytes / 4 - 1;
  static_assert(sizeof(FwdParams) > 256 && sizeof(FwdParams) <= 384, "six lines of 64 bytes");
  const uint32_t x0 = a[0], x1 = a[16], x2 = a[32], x3 = a[48], x4 = a[64], x5 = a[last];
  asm volatile("" ::"s"(x0), "s"(x1), "s"(x2), "s"(x3), "s"(x4), "s"(x5));
}

// Tickets of a table that serves another call (in a trace 5 us, most of it the launch; schedule_rows_kernel 9).
__global__ void clear_tickets_kernel(uint32_t* tickets, int stride) {
  if (threadIdx.x < 8) tickets[(size_t)threadIdx.x * stride] = 0;
}

__global__ void clear_state_kernel(uint64_t* bits, size_t words, unsigned long long* stats, size_t nstats) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t x = i; x < words; x += stride) bits[x] = 0;
  for (size_t x = i; x < nstats; x += stride) stats[x] = 0;
}

// Skip-List of ONE Q-tile row, built by one wave (all 64 lanes call this).  The list is run-length encoded as the
// paper describes: one entry (start | end << 16) per maximal run of consecutive live K/V tiles [start, end), in
// visiting order (ascending, or -- "diagonal first" -- the tiles from the diagonal one to the last, then those before
// the diagonal; a row then has at most floor(Tk/2) + 1 runs).  Lane l looks at bit l of each 64-tile word: a live
// tile whose predecessor is not live starts a run, one whose successor is not live ends it; the k-th start and the
// k-th end of a row belong to the same run, so the two 16-bit halves are written independently at the position
// given by a ballot + prefix popcount.  `extra` (may be null, W words, any address space the caller's lambda reads):
// bits to be OR-ed into the mask row first.  Returns the number of runs in ns and of live tiles in n (same in every
// lane).
template <class ExtraBits>
__device__ __forceinline__ void compact_row(const uint64_t* __restrict__ mrow, ExtraBits extra, int i, int Tk, int W,
                                            int diagonal_first, uint32_t* __restrict__ row_runs, uint32_t& ns,
                                            uint32_t& n) {
  const int lane = threadIdx.x & 63;
  uint16_t* out = reinterpret_cast<uint16_t*>(row_runs);
  uint32_t ne = 0;
  ns = 0;
  n = 0;
  // runs of the live tiles inside [lo, hi), ascending, appended to the list
  auto emit = [&](int lo, int hi) {
    auto live_word = [&](int w) -> uint64_t {  // bit l set = tile 64w+l lies in [lo, hi) and is not skipped
      if (w < 0 || w >= W || 64 * w >= hi || 64 * w + 64 <= lo) return 0ull;
      uint64_t m = ~(mrow[w] | extra(w));
      if (hi - 64 * w < 64) m &= (1ull << (hi - 64 * w)) - 1ull;
      if (lo > 64 * w) m &= ~((1ull << (lo - 64 * w)) - 1ull);
      return m;
    };
    if (hi <= lo) return;
    uint64_t prev = 0ull, cur = live_word(lo >> 6);
    for (int w = lo >> 6; 64 * w < hi; ++w) {
      const uint64_t next = live_word(w + 1);
      const uint64_t starts = cur & ~((cur << 1) | (prev >> 63));
      const uint64_t ends = cur & ~((cur >> 1) | (next << 63));
      const uint64_t below = (1ull << lane) - 1ull;
      const int j = 64 * w + lane;
      if ((starts >> lane) & 1ull) out[2 * (ns + __popcll(starts & below))] = (uint16_t)j;
      if ((ends >> lane) & 1ull) out[2 * (ne + __popcll(ends & below)) + 1] = (uint16_t)(j + 1);
      ns += __popcll(starts);
      ne += __popcll(ends);
      n += __popcll(cur);
      prev = cur;
      cur = next;
    }
  };
  if (diagonal_first) {  // visiting order i, i+1, ..., Tk-1, 0, ..., i-1: the diagonal tile comes first
    const int d = min(i, Tk);
    emit(d, Tk);
    emit(0, d);
  } else {
    emit(0, Tk);
  }
}

// Skip-List compaction as a kernel of its own (the first call of a trajectory, and after the mask was imported;
// otherwise the fused kernel's epilogue has already built the lists of the next call): a wave takes kRowsPerWave
// consecutive rows (Implementation, "Producer and Skip-List Optimization").
__global__ __launch_bounds__(256) void compact_skiplist(const uint64_t* __restrict__ bits, int rows, int Tq, int Tk,
                                                         int W, int diagonal_first, int run_stride,
                                                         uint32_t* __restrict__ runs, uint32_t* __restrict__ nruns,
                                                         uint32_t* __restrict__ live_cnt, uint32_t* heads_ranked) {
  const int lane = threadIdx.x & 63;
  if (blockIdx.x == 0 && threadIdx.x == 0) *heads_ranked = 0;
  const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
  for (int row = wave * kRowsPerWave; row < min(rows, (wave + 1) * kRowsPerWave); ++row) {
    uint32_t ns, n;
    compact_row(bits + (size_t)row * W, [](int) { return 0ull; }, row % Tq, Tk, W, diagonal_first,
                runs + (size_t)row * run_stride, ns, n);
    if (lane == 0) {
      nruns[row] = ns;
      live_cnt[row] = n;
    }
  }
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  f32x2 f = {a, b};
  bf16x2 h = __builtin_convertvector(f, bf16x2);
  return *reinterpret_cast<uint32_t*>(&h);
}

__device__ __forceinline__ float other_half_max(float x) {
  // lanes l and l^32 exchange x; returns max(x, partner's x) in every lane
  const uint32_t u = __float_as_uint(x);
  const u32x2 sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

__device__ __forceinline__ float other_half_sum(float x) {
  const uint32_t u = __float_as_uint(x);
  const u32x2 sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// The row schedule of rows with Skip-Lists.  First half, a workgroup per head: ranks its Q-tile rows by the length of
// their Skip-List, longest first (counting sort, histogram in LDS), and cuts the ranking into chunks of kChunkRows rows
// ("rank c" = rows ranked [c*kChunkRows, (c+1)*kChunkRows)).  The chunks of all heads are numbered rank-major,
// u = c * BH + (h + c) % BH; chunk_work[u] = the chunk's live tiles plus kRowOverhead per row (what a row costs
// besides its tiles, in tile times).  The results go past the L2: a workgroup of another XCD may read them in this launch.
constexpr int kRowOverhead = 2;
__device__ __forceinline__ void rank_head(const RowSchedule& p, int bh, uint32_t* hist) {
  // hist: Tk + 1 bins; bin b counts rows with Tk - b live tiles; then one sum per chunk
  const int Tq = p.Tq, Tk = p.Tk, BH = p.BH, tid = threadIdx.x;
  uint32_t* csum = hist + (Tk + 1);
  const int ranks = (Tq + kChunkRows - 1) / kChunkRows;
  const uint32_t* cnt = p.live_cnt + (size_t)bh * Tq;
  for (int b = tid; b <= Tk + ranks; b += 256) hist[b] = 0;
  __syncthreads();
  for (int i = tid; i < Tq; i += 256) atomicAdd(&hist[Tk - min((int)cnt[i], Tk)], 1u);
  __syncthreads();
  if (tid == 0) {  // exclusive prefix sum over at most 16384 bins
    uint32_t run = 0;
    for (int b = 0; b <= Tk; ++b) {
      const uint32_t c = hist[b];
      hist[b] = run;
      run += c;
    }
  }
  __syncthreads();
  for (int i = tid; i < Tq; i += 256) {
    const uint32_t live = (uint32_t)min((int)cnt[i], Tk);
    const uint32_t pos = atomicAdd(&hist[Tk - live], 1u);
    store_through(p.order + (size_t)bh * Tq + pos, (uint32_t)i);
    atomicAdd(&csum[pos / kChunkRows], live + kRowOverhead);
  }
  __syncthreads();
  for (int c = tid; c < ranks; c += 256) store_through(p.chunk_work + (size_t)c * BH + (bh + c) % BH, csum[c]);
}

// Second half, by the workgroup that has ranked the last head: deals the chunks to the eight XCDs (workgroup id % 8) and
// writes the table the fused kernel reads its row from: slots[x * per_xcd + s] = row of the s-th workgroup of XCD x
// (0xffffffff: none; a chunk always occupies kChunkRows slots, so the chunks of a head's last rank leave some empty);
// xcd_rows[x] = slots in use.  Chunks are taken in the order of u (longest ranks first; consecutive u of a rank belong to
// different heads), each going to the XCD with the least work so far among those holding fewer than per_xcd /
// kChunkRows chunks (the lowest-numbered one on a tie): every XCD ends up with the same work to within about one chunk,
// whatever the number of heads and however the sparsity differs between heads and ranks, and an XCD walks its chunks from
// long rows to short ones.  The workgroups sharing one L2 stream the K/V of the same head (a chunk stays together).
// The greedy pass is serial in the chunks (about 0.1 us each): wave 0 runs it with the state of XCD y in lane y --
// key = work << 3 | y, minimum over the eight lanes by three DPP steps -- for up to kDealMax chunks; with more chunks
// than that (64 per XCD) dealing them round-robin is balanced to within a percent or two and needs no pass at all.
constexpr int kDealMax = 512;
__device__ __forceinline__ uint32_t min_over_8_lanes(uint32_t key) {
  // lanes 8k..8k+7 all end up with the minimum of their eight keys
  key = min(key, (uint32_t)__builtin_amdgcn_update_dpp((int)key, (int)key, 0xB1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
  key = min(key, (uint32_t)__builtin_amdgcn_update_dpp((int)key, (int)key, 0x4E, 0xf, 0xf, false));   // quad_perm 2,3,0,1
  key = min(key, (uint32_t)__builtin_amdgcn_update_dpp((int)key, (int)key, 0x141, 0xf, 0xf, false));  // row_half_mirror
  return key;
}

__device__ __forceinline__ void deal_rows(const RowSchedule& p, uint32_t* work) {
  uint32_t* dest = work + kDealMax;  // work of chunk u; xcd << 29 | first slot of chunk u
  const int BH = p.BH, Tq = p.Tq, chunks = p.chunks, per_xcd = p.per_xcd;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ranks = (Tq + kChunkRows - 1) / kChunkRows;
  const uint32_t cap = (uint32_t)(per_xcd / kChunkRows);  // (the last entry of an XCD's share of the table is its ticket)
  auto through = [](const uint32_t* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  if (tid < 8) p.slots[(size_t)tid * per_xcd + per_xcd - 1] = 0;
  const bool greedy = chunks <= kDealMax;
  if (greedy) {
    for (int u = tid; u < chunks; u += 256) work[u] = through(p.chunk_work + u);
    __syncthreads();
    if (tid < 64) {
      // a chunk's work is below 2^21 (64 rows of at most 16383 + kRowOverhead tiles), an XCD's below 2^27
      uint32_t load = 0, nch = 0, w = work[0];
      for (int u = 0; u < chunks; ++u) {
        const uint32_t w_next = work[min(u + 1, chunks - 1)];  // read ahead: keeps the LDS latency out of the chain
        const uint32_t key = (lane < 8 && nch < cap) ? (load << 3 | (uint32_t)lane) : 0xffffffffu;
        const int best = (int)(__builtin_amdgcn_readfirstlane(min_over_8_lanes(key)) & 7u);
        if (lane == best) {
          dest[u] = ((uint32_t)best << 29) | (nch * kChunkRows);
          load += w;
          nch += 1;
        }
        w = w_next;
      }
      if (lane < 8) p.xcd_rows[lane] = nch * kChunkRows;
    }
    __syncthreads();
  } else if (tid < 8) {  // round-robin: XCD x holds chunks x, x + 8, ...
    p.xcd_rows[tid] = (uint32_t)((chunks - tid + 7) / 8) * kChunkRows;
  }
  // the table: one entry per (head, position in its ranking padded to whole chunks), eight rankings in flight together
  const long long padded = (long long)ranks * kChunkRows, total = (long long)BH * padded;
  constexpr int kAhead = 8;
  for (long long idx0 = tid; idx0 < total; idx0 += 256 * kAhead) {
    uint32_t at[kAhead], row[kAhead];
#pragma unroll
    for (int x = 0; x < kAhead; ++x) {
      const long long idx = idx0 + 256 * x;
      at[x] = 0xffffffffu;
      row[x] = 0xffffffffu;
      if (idx >= total) continue;
      const int bh = (int)(idx / padded), pos = (int)(idx % padded);
      const int c = pos / kChunkRows, u = c * BH + (bh + c) % BH;
      const uint32_t d = greedy ? dest[u] : (((uint32_t)(u & 7) << 29) | (uint32_t)((u >> 3) * kChunkRows));
      const uint32_t s = (d & 0x1fffffffu) + (uint32_t)(pos % kChunkRows);
      if (s < (uint32_t)per_xcd) at[x] = (d >> 29) * (uint32_t)per_xcd + s;
      if (pos < Tq) row[x] = (uint32_t)bh * Tq + through(p.order + (size_t)bh * Tq + pos);
    }
#pragma unroll
    for (int x = 0; x < kAhead; ++x)
      if (at[x] != 0xffffffffu) p.slots[at[x]] = row[x];
  }
}

// Row schedule of a call with short rows (FEW, kFewRows < rows <= kSchedRows), from the mask itself, in one launch:
// workgroup x names the rows of XCD x.  Rows are numbered (head, Q tile); an XCD takes a contiguous range of them -- its
// workgroups share the K/V of a few heads in its L2 -- such that all ranges hold the same work (live tiles +
// kRowOverhead per row).  Where heads differ so much that a range would exceed per_xcd rows, an XCD takes two ranges: an
// eighth, by number, of the rows with at most the mean work, and of the longer ones as many as bring it to an eighth of all
// work (there is always room for some: the first kind holds less than an eighth).  At most 1.9 times its share of
// rows then; should that still be too many, an eighth of the rows in order.  Busiest XCD's work over the mean, from the
// table: 40 heads x 61 tiles, half of the heads 70 % live, half 20 %, 1.32 with the overflow handed to the next XCD,
// 1.005 with two ranges; 90 / 15 % 1.84 -> 1.003; one dense head of eight 2.8 -> 1.03.
// Within its range the longest rows come first, in kLengthClasses classes, heads and Q tiles in order inside a class
// (rows of one head and similar length run side by side).  Every workgroup counts the live tiles of all rows (at most
// three words each).
// Bound by latency: a dozen dependent steps.  With the V^T pass gone it replaces three launches (ranking, dealing,
// transposing; 31 us beside 210-305 us of attention for 888 rows of 37 tiles): three steps of that layer 750 -> 627 us,
// two of 2440 rows x 61 tiles 3850 -> 3661, four of 1320 x 110 (diagonal first) 2262 -> 2165, three of 5120 x 128
// 10040 -> 9918.  At 256 tiles and more the V^T pass is the better bargain again (its cost goes with the tiles, the
// transposing reads' with their square): 3072 x 256 dense 5664 -> 5699, 6000 x 300 20.23 -> 20.53 ms, 2400 x 400 10.98
// -> 11.24 ms.
constexpr int kLengthClasses = 32;
constexpr int kSchedThreads = 1024;
__global__ __launch_bounds__(kSchedThreads) void schedule_rows_kernel(const uint64_t* __restrict__ bits, int rows,
                                                                       int Tk, int W, int per_xcd,
                                                                       uint32_t* __restrict__ slots,
                                                                       uint32_t* __restrict__ xcd_rows) {
  constexpr int kWaves = kSchedThreads / 64;
  // before each thread's piece of the rows: work of the long rows | work of the others << 24 | number of the others << 48
  __shared__ uint64_t part[kSchedThreads];
  static_assert((uint64_t)kSchedRows * (kShortTiles + kRowOverhead) < 1u << 24 && kSchedRows < 1 << 16, "fields of `part`");
  __shared__ uint64_t wave_sum[kWaves];
  __shared__ uint32_t table[kLengthClasses * kWaves];
  __shared__ uint32_t class_base[kLengthClasses];
  // where XCD y's ranges start (9: where the last one ends): row, and rows of the kind before it
  __shared__ int first_long[9], longs_before[9], first_other[9], others_before[9];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, xcd = blockIdx.x;
  auto live_tiles = [&](int row) -> uint32_t {
    uint32_t n = 0;
    for (int w = 0; w < W; ++w) {
      uint64_t m = ~bits[(size_t)row * W + w];
      if (w == W - 1 && (Tk & 63)) m &= (1ull << (Tk & 63)) - 1ull;
      n += (uint32_t)__popcll(m);
    }
    return n;
  };
  const int piece = (rows + kSchedThreads - 1) / kSchedThreads;
  const int lo = min(rows, tid * piece), hi = min(rows, lo + piece);
  uint32_t total = 0;
  uint32_t bar = 0;  // rows of more than bar / rows work count as long: all of them, those above the mean, none
  auto is_long = [&](uint32_t work) { return work * (uint32_t)rows > bar; };
  int l0, l1, o0, o1;  // this XCD's ranges: long rows of [l0, l1), others of [o0, o1)
  const int room = per_xcd - kTableTail;  // for rows
  for (int attempt = 0;; ++attempt) {
    // this thread's contiguous piece, then a scan over the threads
    uint64_t sum = 0;
    for (int r = lo; r < hi; ++r) {
      const uint32_t work = live_tiles(r) + kRowOverhead;
      sum += is_long(work) ? (uint64_t)work : ((uint64_t)work << 24) | (1ull << 48);
    }
    uint64_t scan = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t o = __shfl_up((unsigned long long)scan, d, 64);
      if (lane >= d) scan += o;
    }
    if (lane == 63) wave_sum[wave] = scan;
    __syncthreads();
    uint64_t before = 0, all = 0;
    for (int x = 0; x < kWaves; ++x) {
      if (x < wave) before += wave_sum[x];
      all += wave_sum[x];
    }
    part[tid] = before + scan - sum;
    total = (uint32_t)(all & 0xffffffu) + (uint32_t)((all >> 24) & 0xffffffu);
    const int others = (int)(all >> 48);
    __syncthreads();
    // boundaries: y/8 of the others before the one, of the long rows what completes y/8 of the work before the other
    if (tid < 9) {
      int b = 0, left = others * tid / 8;
      others_before[tid] = left;
      uint32_t other_work = 0;
      if (left > 0) {
        int t = 0;
        for (int step = kSchedThreads / 2; step > 0; step >>= 1)  // last thread with fewer than that before its piece
          if ((int)(part[t + step] >> 48) < left) t += step;
        b = min(rows, t * piece);
        left -= (int)(part[t] >> 48);
        other_work = (uint32_t)(part[t] >> 24) & 0xffffffu;
        for (; b < rows && left > 0; ++b) {
          const uint32_t work = live_tiles(b) + kRowOverhead;
          if (!is_long(work)) {
            other_work += work;
            --left;
          }
        }
      }
      first_other[tid] = b;
      b = rows;
      int longs = rows - others;
      if (tid < 8) {
        const int64_t goal = (int64_t)total * tid - 8 * (int64_t)other_work;  // in eighths
        int t = 0;
        for (int step = kSchedThreads / 2; step > 0; step >>= 1)  // last thread whose piece starts below the goal
          if (8 * (int64_t)(part[t + step] & 0xffffffu) < goal) t += step;
        b = min(rows, t * piece);
        longs = b - (int)(part[t] >> 48);
        int64_t work = (int64_t)(part[t] & 0xffffffu);
        for (; b < rows && 8 * work < goal; ++b) {
          const uint32_t w = live_tiles(b) + kRowOverhead;
          if (is_long(w)) {
            work += w;
            ++longs;
          }
        }
      }
      first_long[tid] = b;
      longs_before[tid] = longs;
    }
    for (int x = tid; x < kLengthClasses; x += kSchedThreads) class_base[x] = 0;
    __syncthreads();
    bool fits = true;
    int start = 0, count = 0;  // (goals a row apart may come out in the other order)
    l0 = l1 = 0;
    for (int y = 1; y <= 8; ++y) {
      const int s = max(start, first_long[y]), c = max(count, longs_before[y]);
      fits = fits && c - count + others_before[y] - others_before[y - 1] <= room;
      if (y == xcd + 1) {
        l0 = start;
        l1 = s;
      }
      start = s;
      count = c;
    }
    o0 = first_other[xcd];
    o1 = first_other[xcd + 1];
    if (fits || attempt == 2) break;  // (an eighth of the rows, by number, always fits: 8 * room >= rows)
    bar = attempt == 0 ? total : 0xffffffffu;
    __syncthreads();
  }
  const int span = l1 - l0, n = span + o1 - o0;  // rows to look at; those of the other kind are passed over
  auto row_at = [&](int x) { return x < span ? l0 + x : o0 + x - span; };
  auto length_class = [&](int x) -> int {
    if (x >= n) return -1;
    const uint32_t live = live_tiles(row_at(x));
    if (is_long(live + kRowOverhead) != (x < span)) return -1;
    return (int)((uint32_t)(Tk - live) * kLengthClasses / (uint32_t)(Tk + 1));
  };
  // class sizes -> first position of each class
  for (int x = tid; x < n; x += kSchedThreads) {
    const int c = length_class(x);
    if (c >= 0) atomicAdd(&class_base[c], 1u);
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t run = 0;
    for (int x = 0; x < kLengthClasses; ++x) {
      const uint32_t c = class_base[x];
      class_base[x] = run;
      run += c;
    }
    xcd_rows[xcd] = run;
  }
  // this XCD's ticket and arrival counters, the marks of the table's calls; before them, whether all rows are of full length,
  // so that some are to be cut
  if (tid < kTableTail)
    slots[(size_t)xcd * per_xcd + per_xcd - 1 - tid] =
        tid == kTableTail - 1 && total == (uint32_t)rows * (uint32_t)(Tk + kRowOverhead) ? 1u : 0u;
  __syncthreads();
  // positions inside the classes, in row order: kSchedThreads rows at a time
  for (int x0 = 0; x0 < n; x0 += kSchedThreads) {
    const int mine = length_class(x0 + tid);
    uint32_t rank = 0;
#pragma unroll 4
    for (int y = 0; y < kLengthClasses; ++y) {
      const uint64_t same = __ballot(mine == y);
      if (mine == y) rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
      if (lane == 0) table[y * kWaves + wave] = (uint32_t)__popcll(same);
    }
    __syncthreads();
    if (mine >= 0) {
      uint32_t pos = class_base[mine] + rank;
      for (int y = 0; y < wave; ++y) pos += table[mine * kWaves + y];
      slots[(size_t)xcd * per_xcd + pos] = (uint32_t)row_at(x0 + tid);
    }
    __syncthreads();
    if (tid < kLengthClasses) {
      uint32_t c = 0;
      for (int y = 0; y < kWaves; ++y) c += table[tid * kWaves + y];
      class_base[tid] += c;
    }
    __syncthreads();
  }
}

// V -> V^T pre-pass.  The PV product contracts over the K/V index, so the matrix cores want, per lane, 8 V values
// of ONE feature d at 8 K/V positions: a 16-byte read from a [d][kv] layout, but a strided gather from V's [kv][d].
// (gfx950's transposing LDS read, ds_read_b64_tr_b16, takes V as it is, at 8 bytes per lane: 16 LDS instructions more per
// stage, the same LDS cycles, 1.8 % of the fused kernel's time, which beyond kShortTiles tiles a row is more than this pass
// costs.)  This kernel writes, once per call,
// vt[bh][d][n_pad] with n_pad = 128 * Tk, zero beyond the sequence, with the K/V index permuted inside every
// group of 16: position 8*h + t holds K/V offset 4*h + t + 4*(t >= 4) -- the order in which a lane of the fused
// kernel holds its P~ values.  One workgroup transposes one 128 x 128 tile through LDS, twice: once with
// transposing reads, once to regroup, because a wave that stores the transposed pieces as it reads them writes 64
// separate 16-byte pieces.  Bound by memory: 55 -> 39 us for 12 heads x 32760 tokens (3.7 -> 5.1 TB/s; a large copy
// reaches 4.9).
// The first workgroups, one per head, make the row schedule: a chain of latencies on a few CUs, hidden behind the
// transposing ones.  As launches of their own its halves took 17 us and two gaps: a late step of 12 heads x 256 tiles 2250 ->
// 2236 us, a dense one 5553 -> 5536.
constexpr int kVtRow = 256 + 16;  // padded LDS row (bytes)
__global__ __launch_bounds__(256) void prepare_rows_kernel(const RowSchedule sched, const uint16_t* __restrict__ v,
                                                            uint16_t* __restrict__ vt, int64_t stride_b, int64_t stride_h,
                                                            int64_t stride_n, int H, int N, int Tk) {
  extern __shared__ __attribute__((aligned(16))) char tile[];
  constexpr int kRow = kVtRow;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x < sched.BH) {
    uint32_t* lds = reinterpret_cast<uint32_t*>(tile);
    rank_head(sched, blockIdx.x, lds);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the ranking is past the L2 before it is counted)
    __syncthreads();
    if (tid == 0) lds[0] = atomicInc(sched.heads_ranked, (unsigned)sched.BH - 1);
    __syncthreads();
    const bool last = lds[0] == (uint32_t)sched.BH - 1;
    __syncthreads();
    if (last) deal_rows(sched, lds);
    return;
  }
  const int block = blockIdx.x - sched.BH;
  const int j = block % Tk, bh = block / Tk;
  const uint16_t* vb = v + (int64_t)(bh / H) * stride_b + (int64_t)(bh % H) * stride_h;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int r = (tid >> 4) + 16 * t, row = j * 128 + r;
    uint4 x = {0u, 0u, 0u, 0u};
    if (row < N) x = *reinterpret_cast<const uint4*>(vb + (int64_t)row * stride_n + 8 * (tid & 15));
    *reinterpret_cast<uint4*>(tile + r * kRow + 16 * (tid & 15)) = x;
  }
  __syncthreads();
  const int g = lane >> 4, i16 = lane & 15, r_src = i16 >> 2, c_src = lane & 3;
  uint16_t* out = vt + (int64_t)bh * 128 * (128 * (int64_t)Tk) + (int64_t)j * 128;
  s16x8 o[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int q = 8 * wave + x;                    // 32 (16-group, half, d-half) combinations per tile
    const int c16 = q >> 2, hh = (q >> 1) & 1, dhalf = q & 1;
    const char* src = tile + (16 * c16 + 4 * hh + r_src) * kRow + 2 * (64 * dhalf + 16 * g + 4 * c_src);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LA_LDS s16x4*)(src));
    const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LA_LDS s16x4*)(src + 8 * kRow));
    o[x] = __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  __syncthreads();
  // back through LDS as [d][kv], so that 16 lanes store a whole 256-byte piece of a feature row
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int q = 8 * wave + x, d = 64 * (q & 1) + 16 * g + i16;
    *reinterpret_cast<s16x8*>(tile + d * kRow + 32 * (q >> 2) + 16 * ((q >> 1) & 1)) = o[x];
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int d = (tid >> 4) + 16 * t;
    *reinterpret_cast<uint4*>(out + (int64_t)d * (128 * (int64_t)Tk) + 8 * (tid & 15)) =
        *reinterpret_cast<const uint4*>(tile + d * kRow + 16 * (tid & 15));
  }
}

// The live K/V tiles of one Skip-Mask row in visiting order, walked from the mask words themselves (calls with few or
// short rows, where a list built by an earlier kernel would cost more than it saves): lane w of the wave holds word w
// of the row's live set, the position is scalar.  Rows of at most 64 words (4096 tiles).  Used by whole waves only.
struct LiveWalk {
  uint32_t lo, hi;   // this lane's word of the live set
  int W, start;      // words of a row; tile the visit starts with (diagonal first: the diagonal tile)
  int v;             // visit position: the words from the starting one on, cyclically (the starting one twice: its tiles
                     // from `start` on first, those before it last)
  uint64_t cur;      // tiles of the current word still to come

  // Lanes past the row, and all of them for an empty mask, lie past the end of the buffer and read zeros: with a branch
  // around it the load was waited for before the Q loads behind it were issued (options clip, four steps, 198 -> 195 us).
  static __device__ __forceinline__ uint64_t load(const uint64_t* mrow, bool empty_mask, int words) {
    const auto at = __builtin_amdgcn_make_buffer_rsrc((void*)mrow, 0, empty_mask ? 0 : 8 * words, 0x00020000);
    return __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(at, 8 * (int)(threadIdx.x & 63), 0, 0));
  }
  __device__ __forceinline__ void open(uint64_t skipped, int Tk, int W_, int start_) {
    const int lane = threadIdx.x & 63;
    W = W_;
    start = start_;
    uint64_t live = 0;
    if (lane < W) {
      live = ~skipped;
      if (lane == W - 1 && (Tk & 63)) live &= (1ull << (Tk & 63)) - 1ull;
    }
    lo = (uint32_t)live;
    hi = (uint32_t)(live >> 32);
    rewind();
  }
  __device__ __forceinline__ int words() const { return start > 0 ? W + 1 : W; }
  __device__ __forceinline__ int index(int at) const {  // word of visit position `at`
    const int w = (start >> 6) + at;
    return w >= W ? w - W : w;
  }
  __device__ __forceinline__ uint64_t word(int at) const {
    const int w = index(at);
    const uint64_t x =
        (uint32_t)__builtin_amdgcn_readlane(lo, w) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, w) << 32);
    const uint64_t lead = ~0ull << (start & 63);
    return at == 0 ? x & lead : at == W ? x & ~lead : x;
  }
  __device__ __forceinline__ void rewind() {
    v = 0;
    cur = word(0);
  }
  __device__ __forceinline__ void count(int& tiles, int& runs) const {  // of the whole row
    tiles = 0;
    runs = 0;
    uint64_t prev = 0;
    for (int at = 0; at < words(); ++at) {
      const uint64_t x = word(at);
      if (index(at) == 0) prev = 0;  // a run does not continue from the last tile to the first
      tiles += __popcll(x);
      runs += __popcll(x & ~((x << 1) | (prev >> 63)));
      prev = x;
    }
  }
  __device__ __forceinline__ void skip(int n) {  // n tiles ahead; n is less than the tiles left
    while (v + 1 < words()) {
      const int c = __popcll(cur);
      if (c > n) break;
      n -= c;
      cur = word(++v);
    }
    for (; n > 0; --n) cur &= cur - 1;
  }
  __device__ __forceinline__ bool next(int& j) {  // the next tile; false (j unchanged) at the end
    while (cur == 0 && v + 1 < words()) cur = word(++v);
    if (cur == 0) return false;
    j = 64 * index(v) + __builtin_ctzll(cur);
    cur &= cur - 1;
    return true;
  }
};

// Geometry of the fused kernel: a wave owns QB blocks of 32 Q rows, a workgroup (one Q tile of 128 rows) has 4/QB waves.
template <int QB>
struct Geo {
  static constexpr int kWaves = 4 / QB;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kChunks = 16 / kWaves;  // 1 KB DMA pieces of a K (or V) stage per wave
};

// Per-lane constants of the fused kernel.
template <int QB>
struct Lane {
  u32x4 krsrc, vrsrc;  // buffer descriptors of this head's K (range-checked: rows past the end read as 0) and V^T
  uint32_t kdma[Geo<QB>::kChunks], vdma[Geo<QB>::kChunks];  // byte offsets (inside a stage) of this lane's DMA pieces
  uint32_t kread[8];  // LDS address of the K fragment for d-chunk kk in stage buffer 0 (stage and block: immediates)
  uint32_t vread[4];  // LDS address of the V^T fragment for column chunk cc in buffer 0 (d-block via immediates)
  uint32_t lds_wave;  // LDS address of this wave's first DMA piece inside stage buffer 0 (wave-uniform)
  uint32_t stride2;   // stride_n * 2 (bytes per token row)
  int hi;
  int col;            // PAIR: first column of this group's half of a tile (wave-uniform)
  bool qvalid[QB];
  float c;            // scale * log2(e)
  float scale, thr;
  int N;
};

template <int QB, bool IMM>
struct State {
  bf16x8 qf[QB][8];
  f32x16 oacc[QB][4];
  f32x16 sA[QB][2], sB[QB][2];  // S^T of even / odd stages
  uint32_t pw[QB][16];          // P~^T of the previous stage, bf16 pairs; words 4cc..4cc+3 = B operand of chunk cc
                                // (IMM: of the previous odd stage)
  uint32_t pw0[QB][16];         // IMM only: P~^T of the previous even stage
  float m_run[QB], l_run[QB], mloc_tile[QB];
  // IMM only: row sum of the tile in flight (added to l_run once the tile is known not to have fired), and the
  // rescale factor of the previous stage, which O^T has not seen yet because its PV product runs a stage later
  // (PAIR: of the two tiles in flight, by parity)
  float l_pend[QB][2], alpha_prev[QB];
  bool grew_prev;
  // PAIR only: this wave's row maxima of the previous tile (its half of the columns), and the running row maximum over
  // both halves
  float mloc_prev, m_all;
};

// Buffer descriptor (V#) of a raw buffer of `bytes` bytes at `ptr`: loads at offsets >= bytes return zero.
__device__ __forceinline__ u32x4 make_rsrc(const void* ptr, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(ptr);
  u32x4 r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
  return r;
}

// Descriptor of the same buffer seen from `off` bytes in (wave-uniform, scalar arithmetic): base += off, size -= off
// (0 if off is past the end, so that every load through it returns zeros).  Folding the moving part of a DMA address
// into the descriptor leaves the per-lane offsets loop-invariant: no vector add per load.
__device__ __forceinline__ u32x4 rebase(const u32x4 r, uint32_t off) {
  off = __builtin_amdgcn_readfirstlane(off);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(r[0]), hi = __builtin_amdgcn_readfirstlane(r[1]);
  const uint32_t size = __builtin_amdgcn_readfirstlane(r[2]);
  // base += off (the high word holds only address bits here: stride and swizzle fields are zero); size =
  // max(size - off, 0).  Four scalar instructions; the compiler's own 64-bit add and saturating subtract take ten.
  uint32_t nlo, nhi, left;
  asm("s_add_u32 %0, %3, %5\n\ts_addc_u32 %1, %4, 0\n\ts_sub_u32 %2, %6, %5\n\ts_cselect_b32 %2, 0, %2"
      : "=&s"(nlo), "=&s"(nhi), "=&s"(left)
      : "s"(lo), "s"(hi), "s"(off), "s"(size)
      : "scc");
  u32x4 o = {nlo, nhi, left, (uint32_t)__builtin_amdgcn_readfirstlane(r[3])};
  return o;
}

// One 1 KB piece global -> LDS without registers: lane l's 16 bytes land at lds_addr + 16*l.  Written as inline
// assembly so that the compiler does not order later LDS reads of OTHER buffers behind this load (it would wait
// for vmcnt(0) before every LDS read); completion is enforced by the s_waitcnt vmcnt(0) + barrier ending a stage.
// (Issuing a stage's four pieces of K or V back to back with one M0 update -- their LDS offsets riding in the
// instruction offset -- was measured 3-6 % slower on the dense step: a burst of memory instructions holds up the
// MFMA behind it.)
// LDS address = lds_base (a wave-uniform register) + kLdsOff (a compile-time constant added on the scalar unit, so
// that the sixteen destinations of a stage pair do not each occupy a scalar register across the main loop).
template <int kLdsOff>
__device__ __forceinline__ void dma16(const u32x4 rsrc, uint32_t lds_base, uint32_t voffset) {
  asm volatile("s_add_u32 m0, %2, %3\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(voffset), "s"(rsrc), "s"(lds_base), "n"(kLdsOff)
               : "memory", "m0", "scc");
}

template <int QB, int kBufOff, int X = 0>
__device__ __forceinline__ void dma_stage(const u32x4 rsrc, const uint32_t* off, uint32_t stage_byte_base,
                                          uint32_t lds_wave_addr) {
  if constexpr (X < Geo<QB>::kChunks) {
    dma16<kBufOff + 1024 * X>(rsrc, lds_wave_addr, off[X] + stage_byte_base);
    dma_stage<QB, kBufOff, X + 1>(rsrc, off, stage_byte_base, lds_wave_addr);
  }
}

// Piece x (compile-time after unrolling) of a stage: dispatch to the instance with that LDS offset.
template <int QB, int kBufOff>
__device__ __forceinline__ void dma_piece(int x, const u32x4 rsrc, const uint32_t* off, uint32_t stage_byte_base,
                                          uint32_t lds_wave_addr) {
  switch (x) {
    case 0: dma16<kBufOff + 0 * 1024>(rsrc, lds_wave_addr, off[0] + stage_byte_base); break;
    case 1: dma16<kBufOff + 1 * 1024>(rsrc, lds_wave_addr, off[1] + stage_byte_base); break;
    case 2: dma16<kBufOff + 2 * 1024>(rsrc, lds_wave_addr, off[2] + stage_byte_base); break;
    case 3: dma16<kBufOff + 3 * 1024>(rsrc, lds_wave_addr, off[3] + stage_byte_base); break;
    case 4: dma16<kBufOff + 4 * 1024>(rsrc, lds_wave_addr, off[4 % Geo<QB>::kChunks] + stage_byte_base); break;
    case 5: dma16<kBufOff + 5 * 1024>(rsrc, lds_wave_addr, off[5 % Geo<QB>::kChunks] + stage_byte_base); break;
    case 6: dma16<kBufOff + 6 * 1024>(rsrc, lds_wave_addr, off[6 % Geo<QB>::kChunks] + stage_byte_base); break;
    default: dma16<kBufOff + 7 * 1024>(rsrc, lds_wave_addr, off[7 % Geo<QB>::kChunks] + stage_byte_base); break;
  }
}

__device__ __forceinline__ bf16x8 p_operand(const uint32_t* w) {
  const u32x4 v = {w[0], w[1], w[2], w[3]};
  return __builtin_bit_cast(bf16x8, v);
}

// S^T(next) = K Q^T for one 64-column stage held in LDS at byte offset sK (kread: absolute addresses in buffer 0).
template <int QB>
__device__ __forceinline__ void mma_qk(f32x16 (&nxt)[QB][2], const bf16x8 (&qf)[QB][8], int sK,
                                       const uint32_t (&kread)[8]) {
#pragma unroll
  for (int blk = 0; blk < 2; ++blk) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int r = 0; r < 16; ++r) nxt[qb][blk][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const bf16x8 a = *reinterpret_cast<LA_LDS const bf16x8*>(kread[kk] + (uint32_t)(sK + 8192 * blk));
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        nxt[qb][blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[qb][kk], nxt[qb][blk], 0, 0, 0);
    }
  }
}

// V fragment of 16 K/V positions x 32 features (column chunk cc, d-block db) from a V stage as it lies in memory ([kv][d]):
// two transposing reads, rows 4h..4h+3 and 8+4h..8+4h+3 of the chunk for lane half h -- the order of the P~ values.
__device__ __forceinline__ bf16x8 load_v_rows(uint32_t addr) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LA_LDS s16x4*)(addr));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LA_LDS s16x4*)(addr + 8 * 256));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// O^T += V^T P~^T for one 64-column stage held in LDS at byte offset sV ([d][64 kv], 128-byte rows).
template <int QB, bool VROWS>
__device__ __forceinline__ void mma_pv(f32x16 (&oacc)[QB][4], const uint32_t (&pw)[QB][16], int sV,
                                       const uint32_t (&vread)[4]) {
#pragma unroll
  for (int cc = 0; cc < 4; ++cc)
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      bf16x8 a;
      if constexpr (VROWS)
        a = load_v_rows(vread[db] + (uint32_t)(sV + 4096 * cc));
      else
        a = *reinterpret_cast<LA_LDS const bf16x8*>(vread[cc] + (uint32_t)(sV + 4096 * db));
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        oacc[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p_operand(&pw[qb][4 * cc]), oacc[qb][db], 0, 0, 0);
    }
}

// LDS -> register fragment k of a stage's matrix work: k < 16 is the V^T fragment (column chunk k/4, d-block k%4)
// of O^T += V^T P~^T, k >= 16 the K fragment (block (k-16)/8, d-chunk (k-16)%8) of S^T(s+1) = K Q^T.  Block 1 starts
// only at step 24, after the softmax has consumed block 1 of the current stage: its accumulators reuse those
// registers (alternating the two blocks was measured: no faster, six registers more).
// kread / vread hold absolute LDS addresses (of stage buffer 0), kK / kV are the byte offsets of the stage buffers
// read: every fragment address is one loop-invariant register plus an immediate.
// step k >= 16 of a stage multiplies d-chunk qk_kk(k) of K block qk_blk(k): block 0 first, then block 1
// (alternating the blocks, so that consecutive MFMAs share their Q fragment, measured 0.3 % faster for 4 more registers)
__device__ __forceinline__ constexpr int qk_blk(int k) { return (k - 16) >> 3; }
__device__ __forceinline__ constexpr int qk_kk(int k) { return k & 7; }

template <bool VROWS, int kK, int kV>
__device__ __forceinline__ bf16x8 load_frag(int k, const uint32_t (&kread)[8], const uint32_t (&vread)[4]) {
  if (k >= 16) return *reinterpret_cast<LA_LDS const bf16x8*>(kread[qk_kk(k)] + (uint32_t)(kK + 8192 * qk_blk(k)));
  const int cc = k >> 2, db = k & 3;
  if constexpr (VROWS) return load_v_rows(vread[db] + (uint32_t)(kV + 4096 * cc));
  return *reinterpret_cast<LA_LDS const bf16x8*>(vread[cc] + (uint32_t)(kV + 4096 * db));
}

// Row maximum before the first tile: below every score of finite operands, and finite itself, so that a column half without
// valid columns weighs exp2(-inf - kNoMax c) = 0.
constexpr float kNoMax = -3.402823466e38f;
constexpr int kPrefetch = 3;  // LDS fragments in flight ahead of the MFMA that consumes them
constexpr int kDmaGap = 2;    // steps between two DMA issues of a stage

// One pipeline stage (64 K/V columns).  H = stage parity (half of the mask tile); j_tail = index of the ragged last
// tile of the sequence, whose columns past the end must be masked (-1 if the sequence ends on a tile boundary).
//
// The stage is written as 32 steps.  Step k issues the MFMA(s) of fragment k -- first the 16 of
// O^T += V^T(s-1) P~^T(s-1), then the 16 of S^T(s+1) -- and one slice of the online softmax of stage s (vector
// ALU), with scheduling fences between steps so that the compiler keeps this interleaving: the matrix cores and
// the vector ALU of the SIMD then work at the same time inside one wave.  P~ of stage s is written over P~ of
// stage s-1 word by word, each word after the last MFMA that reads it has been issued.
//
// IMM: the PV product of this stage is that of stage s-2 (same parity: its P~ and V^T buffers are those of parity
// H), issued only if pv_on (wave-uniform: the tile it belongs to did not fire); the V^T stage loaded here is that of
// stage s-1 (tile j_v, the other half), into the buffer of the other parity.
struct NoOp {
  template <class... A>
  __device__ __forceinline__ void operator()(A...) const {}
};

// verdict_load / verdict_commit (first stage of a tile, deferred marking only): the combine of the PREVIOUS tile's four
// per-wave predicate results, spread over this stage -- its LDS read is issued at step 0 and used at step 12, so that
// the wave that does it never waits for it.
// PAIR: a stage is this group's half of a whole tile (H = parity of the tile, j_nxt = the tile two ahead, j_v the
// previous one); verdict_end receives the half's row maxima at the end of the stage.
template <int QB, int H, bool IMM, bool VROWS, bool PAIR, class VLoad = NoOp, class VCommit = NoOp, class VEnd = NoOp>
__device__ __forceinline__ void stage(State<QB, IMM>& st, const Lane<QB>& ln, char* smem, int j_cur, int j_nxt,
                                      int* flag_slot, int j_tail, int j_v = 0, bool pv_on = true,
                                      VLoad verdict_load = VLoad(), VCommit verdict_commit = VCommit(),
                                      VEnd verdict_end = VEnd()) {
  f32x16(&cur)[QB][2] = H ? st.sB : st.sA;
  f32x16(&nxt)[QB][2] = H ? st.sA : st.sB;
  uint32_t(&pwc)[QB][16] = (IMM && !H) ? st.pw0 : st.pw;

  // ---- DMA: K of stage s+2 (next tile, same half) and V of this stage go into the buffers of parity H; the
  // loads are issued one at a time between the steps below (kDmaGap steps apart) so that a full memory
  // instruction queue does not hold up the MFMAs behind it ----
  const int col = PAIR ? ln.col : H * kSub, col_v = PAIR ? ln.col : IMM ? (H ^ 1) * kSub : H * kSub;
  const u32x4 krs = rebase(ln.krsrc, (uint32_t)(j_nxt * kTile + col) * ln.stride2);
  const u32x4 vrs = rebase(ln.vrsrc, (uint32_t)((IMM ? j_v : j_cur) * kTile + col_v) * (VROWS ? ln.stride2 : 2u));
  constexpr int kVDst = kVOff + (IMM ? (H ^ 1) : H) * kStageBytes;  // V^T buffer the DMA of this stage fills
  constexpr int kC = Geo<QB>::kChunks;

  constexpr int kKSrc = kKOff + (H ^ 1) * kStageBytes;                // K stage read by S^T(s+1)
  constexpr int kVSrc = kVOff + (IMM ? H : (H ^ 1)) * kStageBytes;    // V^T stage read by the PV product
  bf16x8 frag[kPrefetch];
#pragma unroll
  for (int k = 0; k < kPrefetch; ++k)
    if (!IMM || pv_on) frag[k] = load_frag<VROWS, kKSrc, kVSrc>(k, ln.kread, ln.vread);

  float pm[QB], mx[QB], m_new[QB], mc[QB], alpha[QB], lsum[QB], ta0[QB], ta1[QB], tb0[QB], tb1[QB];
  uint32_t wb[QB];  // (kPackLate) packed pair whose sum is still to be taken
  bool ok = true, grew = false;
  // The ragged last tile of the sequence: its columns past the end leave the row maxima and sums (one scalar compare
  // and branch per stage, taken for one tile per row at most).  This lane's element r of block blk is column
  // 32*blk + 8*(r>>2) + (r&3) + 4*hi of the stage: the lane-independent part is compared with one per-lane limit.
  if (j_cur == j_tail) {
    int lim = ln.N - (j_cur * kTile + col) - 4 * ln.hi;
    asm volatile("" : "+v"(lim));  // keeps the compares inside this branch (else their lane masks are formed ahead of
                                   // time, for every stage, and held in scalar registers)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (32 * blk + 8 * (r >> 2) + (r & 3) >= lim) cur[qb][blk][r] = -INFINITY;
          asm volatile("" : "+v"(cur[qb][blk][r]));  // one lane mask alive at a time
        }
  }
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) wb[qb] = 0u;
  constexpr bool kPackLate = VROWS && !IMM;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  auto mfma_part = [&](auto kc, auto qbc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;  // the step index is a compile-time constant: every register index is static
    constexpr int qb = decltype(qbc)::value;
    // ---- matrix cores ----
    const bf16x8 a = frag[k % kPrefetch];
    if (k >= 16) {
      const int blk = qk_blk(k), kk = qk_kk(k);
      {
        if (kk == 0) {
          const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          nxt[qb][blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, st.qf[qb][kk], zero, 0, 0, 0);
        } else {
          nxt[qb][blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, st.qf[qb][kk], nxt[qb][blk], 0, 0, 0);
        }
      }
    } else {
      const int cc = k >> 2, db = k & 3;
      if (!IMM || pv_on)
        st.oacc[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p_operand(&pwc[qb][4 * cc]), st.oacc[qb][db],
                                                                  0, 0, 0);
    }
  };
  auto mem_part = [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    if (k + kPrefetch < 32) {
      if (!IMM || pv_on || k + kPrefetch >= 16)
        frag[k % kPrefetch] = load_frag<VROWS, kKSrc, kVSrc>(k + kPrefetch, ln.kread, ln.vread);
    }
    if (k % kDmaGap == 0 && k / kDmaGap < 2 * kC) {
      const int x = k / kDmaGap;
      if (x < kC)
        dma_piece<QB, kVDst>(x, vrs, ln.vdma, 0u, ln.lds_wave);
      else
        dma_piece<QB, kKOff + H * kStageBytes>(x - kC, krs, ln.kdma, 0u, ln.lds_wave);
    }
    if (k == 0) verdict_load();
  };
  auto vector_part = [&](auto kc, auto qbc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    constexpr int qb = decltype(qbc)::value;
    constexpr int pend = PAIR ? H : 0;
    // ---- vector ALU: slice k of the online softmax of stage s (raw dot products; 1/sqrt(d) folded into c) ----
    {
      if (k < 4) {
        // m_local: this lane's 32 scores in one chain, two more per instruction; four chains of eight take two instructions
        // more to join (vector instructions besides the MFMAs, per MFMA, 40 heads x 591 tiles: 4.38 -> 4.31).  With that and
        // the predicate below in lane masks 12 heads x 256 tiles 5639 -> 5573 us, 40 x 591, two steps, 162.0 -> 161.0 ms, 24 x
        // 931 239.7 -> 238.9: every long layer a little faster, none by more than two runs of one side differ
        const int e0 = k == 0 ? 1 : 8 * k + 1, e1 = k == 3 ? 32 : 8 * k + 9;
        float v = k == 0 ? cur[qb][0][0] : pm[qb];
#pragma unroll
        for (int e = e0; e < e1; ++e) v = fmaxf(v, cur[qb][e >> 4][e & 15]);
        asm volatile("" : "+v"(v));
        pm[qb] = v;
      } else if (k == 4) {
        mx[qb] = other_half_max(pm[qb]);
      } else if (k == 5) {  // m_ij = max(m_{i,j-1}, m_local) and the rescale factor of the earlier stages
        if (!PAIR) st.mloc_tile[qb] = H ? fmaxf(st.mloc_tile[qb], mx[qb]) : mx[qb];
        // the reference of the exponentials is the running maximum itself, at every stage: a row's largest weight is then
        // exactly 1, which bf16 holds without error (a reference trailing the maximum saved 1.5 % of the dense 12-head
        // step and let that rounding error in: up to 9e-3 of the values where large terms cancel)
        m_new[qb] = fmaxf(st.m_run[qb], mx[qb]);
        alpha[qb] = __builtin_amdgcn_exp2f((st.m_run[qb] - m_new[qb]) * ln.c);
        grew = grew || (m_new[qb] > st.m_run[qb]);
        st.m_run[qb] = m_new[qb];
        mc[qb] = m_new[qb] * ln.c;
        lsum[qb] = 0.f;
      } else if (k < 30) {
        // P~ = exp(S - m_ij), packed to bf16: 16 pairs of scores over 24 steps, four vector instructions per step
        // (a cycle of three steps does two pairs: exp exp | pack+sum, exp | exp, pack+sum).  kPackLate: the second pair
        // is packed in the next cycle (exp, pack | exp, sum, exp | pack, exp, sum), so that no instruction directly
        // follows the exponential it uses, which costs a wait state: 0.6 % of the short clip's, the two-layer and the
        // diagonal-first sequence.  Of the others nothing certain is known (long rows: 12 heads dense 0.7 % faster with it,
        // long video 0.45 % slower; immediate pair 0.2 % slower; builds of one source differ by 0.1-0.5 %): they keep the
        // order they had.
        const int t = k - 6, c = t / 3, ph = t % 3;
        const int eA = 2 * c, eB = 2 * c + 1;
        if (kPackLate) {
          auto exponent = [&](int e, int half) {
            return __builtin_fmaf(cur[qb][e >> 3][2 * (e & 7) + half], ln.c, -mc[qb]);
          };
          if (ph == 0) {
            ta0[qb] = __builtin_amdgcn_exp2f(exponent(eA, 0));
            ta1[qb] = exponent(eA, 1);
            if (c > 0) wb[qb] = pack_bf16x2(tb0[qb], tb1[qb]);
            asm volatile("" : "+v"(ta0[qb]), "+v"(ta1[qb]), "+v"(wb[qb]));
            if (c > 0) pwc[qb][eA - 1] = wb[qb];
          } else if (ph == 1) {
            ta1[qb] = __builtin_amdgcn_exp2f(ta1[qb]);
            if (c > 0) lsum[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, wb[qb]), ones, lsum[qb], false);
            tb0[qb] = __builtin_amdgcn_exp2f(exponent(eB, 0));
            asm volatile("" : "+v"(ta1[qb]), "+v"(lsum[qb]), "+v"(tb0[qb]));
          } else {
            uint32_t w = pack_bf16x2(ta0[qb], ta1[qb]);
            tb1[qb] = __builtin_amdgcn_exp2f(exponent(eB, 1));
            lsum[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, lsum[qb], false);
            asm volatile("" : "+v"(w), "+v"(lsum[qb]), "+v"(tb1[qb]));
            pwc[qb][eA] = w;
          }
        } else if (ph == 0) {
          ta0[qb] = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[qb][eA >> 3][2 * (eA & 7)], ln.c, -mc[qb]));
          ta1[qb] = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[qb][eA >> 3][2 * (eA & 7) + 1], ln.c, -mc[qb]));
          // empty volatile asms pin every slice to its step: without them the compiler sinks all the exponentials
          // behind the last MFMA, where nothing overlaps them
          asm volatile("" : "+v"(ta0[qb]), "+v"(ta1[qb]));
        } else if (ph == 1) {
          uint32_t w = pack_bf16x2(ta0[qb], ta1[qb]);
          // the row sum adds the bf16-rounded weights, the same values the PV product uses
          lsum[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, lsum[qb], false);
          tb0[qb] = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[qb][eB >> 3][2 * (eB & 7)], ln.c, -mc[qb]));
          asm volatile("" : "+v"(w), "+v"(lsum[qb]), "+v"(tb0[qb]));
          pwc[qb][eA] = w;  // word e belongs to chunk e/4, whose last reader was the MFMA of step 4*(e/4)+3 < k
        } else {
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[qb][eB >> 3][2 * (eB & 7) + 1], ln.c, -mc[qb]));
          uint32_t w = pack_bf16x2(tb0[qb], p1);
          lsum[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, lsum[qb], false);
          asm volatile("" : "+v"(w), "+v"(lsum[qb]));
          pwc[qb][eB] = w;
        }
      } else if (k == 30) {
        if (kPackLate) {
          wb[qb] = pack_bf16x2(tb0[qb], tb1[qb]);
          lsum[qb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, wb[qb]), ones, lsum[qb], false);
          asm volatile("" : "+v"(wb[qb]), "+v"(lsum[qb]));
          pwc[qb][15] = wb[qb];
        }
        if (!IMM) {
          st.l_run[qb] = st.l_run[qb] * alpha[qb] + lsum[qb];
        } else {
          st.l_run[qb] *= alpha[qb];
          if (PAIR) st.l_pend[qb][H ^ 1] *= alpha[qb];
          st.l_pend[qb][pend] = (!PAIR && H) ? st.l_pend[qb][0] * alpha[qb] + lsum[qb] : lsum[qb];
        }
        if (!PAIR && H) {  // skip predicate of the whole 128-column tile, once its second half is in (eq. sparge_cond)
          const float g = (st.mloc_tile[qb] - m_new[qb]) * ln.scale;  // this row; max over rows = ballot below
          ok = ok && g <= (ln.qvalid[qb] ? ln.thr : INFINITY);
        }
      }
    }
    if (PAIR && k == 30) verdict_end(mx[qb]);
    if (!PAIR && H && k == 31 && qb == QB - 1)
      *flag_slot = __all(ok) ? 1 : 0;  // lane 0: the wave's slot; other lanes: a dummy word each
    if (k == 12 && qb == QB - 1) verdict_commit();
  };
  static_for(std::make_integer_sequence<int, 32>{}, [&](auto kc) __attribute__((always_inline)) {
    // matrix instruction and the memory instructions of the step first, then (fenced) the vector slice: measured
    // 1-1.5 % faster than leaving the order inside a step to the compiler (the memory instructions behind the vector
    // slice was the slowest order tried).  Issuing the MFMAs of 2, 4 or 8 steps back to back before their slices
    // (a coarser ping-pong between the two waves of a SIMD) was measured 0 / 2.5 / 6 % slower.
    static_for(std::make_integer_sequence<int, QB>{}, [&](auto qbc) __attribute__((always_inline)) {
      mfma_part(kc, qbc);
      if (decltype(qbc)::value == 0) mem_part(kc);
      __builtin_amdgcn_sched_barrier(0);
      vector_part(kc, qbc);
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  // O^T of the earlier stages is rescaled after this stage's PV MFMAs (rare once the running max has settled).
  // IMM: O^T now holds the products up to stage s-2 and moves to the reference maximum of stage s-1, whose product
  // the next stage adds; this stage's own factor waits one stage.
  if (IMM ? st.grew_prev : (bool)__any(grew)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.oacc[qb][db][r] *= IMM ? st.alpha_prev[qb] : alpha[qb];
  }
  if (IMM) {
    st.grew_prev = __any(grew);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) st.alpha_prev[qb] = alpha[qb];
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// a / b of small wave-uniform numbers (0 <= a <= 2^23, b >= 1): the rounded reciprocal's product is off by one at most
__device__ __forceinline__ int quotient(int a, int b) {
  int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
  q -= q * b > a;
  q += (q + 1) * b <= a;
  return __builtin_amdgcn_readfirstlane(q);
}

// First visiting position of segment s of a row with cnt live tiles.
__device__ __forceinline__ int segment_start(int cnt, int s, int nseg) {
  return nseg == 1 ? cnt * s : quotient(cnt * s, nseg);
}

// How many places XCD x's list of rows has, and the row at place t of it (-1: none; FEW: the piece of it above kPieceShift).
template <bool FEW>
__device__ __forceinline__ int places_of(const FwdParams& p, int x, int cut) {
  if (!FEW) return (int)p.xcd_rows[x];
  if (p.rows_total > kSchedRows) return p.per_xcd;
  const int share = (p.rows_total + 7) / 8, extra = cut * (p.cut_pieces - 1);
  return (p.scheduled && cut == 0 ? (int)p.xcd_rows[x] : max(0, min(share, p.rows_total - x * share))) + extra;
}
constexpr int kPieceShift = 24;  // (there are at most 2^23 rows without lists)
static_assert(kMaxListless <= 1 << (kPieceShift - 1), "row and piece in one word");
template <bool FEW>
__device__ __forceinline__ int row_at_place(const FwdParams& p, int x, int t, int cut) {
  const int places = places_of<FEW>(p, x, cut);
  if (t >= places) return -1;
  if (!FEW) return (int)p.slots[(size_t)x * p.per_xcd + t];  // (-1 behind a chunk of fewer than kChunkRows)
  if (p.rows_total > kSchedRows) {
    const int row = dealt_chunk(t / kDealtRows, x) * kDealtRows + t % kDealtRows;
    return row < p.rows_total ? row : -1;
  }
  // from the table, or in order, an eighth of the rows to every XCD; of each eighth by number the last `cut` rows in
  // cut_pieces pieces each, of which all but the first end the list, row-fastest
  const int share = (p.rows_total + 7) / 8, rows = places - cut * (p.cut_pieces - 1);
  if (t < rows) return p.scheduled && cut == 0 ? (int)p.slots[(size_t)x * p.per_xcd + t] : x * share + t;
  const int index = quotient(t - rows, cut), row = x * share + share - cut + t - rows - index * cut;
  return row < p.rows_total ? row | (index + 1) << kPieceShift : -1;
}

// The next row for a workgroup that starts on XCD `home` after the first round, by one thread: the next place of its
// own XCD's list; if that list is used up, of the one with most places left; -1 if there are none.  Places below
// kResident belong to the first round's workgroups, which need no counter.  Ends: a draw that fails has found its list
// used up, which it then stays.  Why: workgroups go to XCDs by id, but equal lists do not end together, because the
// XCDs' clocks differ (a tile took 3.2 us on the fastest, 3.6 on the slowest, the same ones in every kernel of a
// session; lists of the 12-head dense step ended between 5.14 and 5.68 ms).  A row drawn costs a counter's round trip
// (0.35 us; kDrawTiles).  Lists by place -> drawn: 40 heads x 591 tiles, dense + sparse step, 170.7 -> 164.8 ms; 24 x
// 931 253.8 -> 245.4; a sparse step of 12 x 256 2379 -> 2331 us; 12 x 110, diagonal first, four steps 2128 -> 2102; no
// gain where few rounds of equally long rows leave nothing to draw (12 x 256 dense, six rounds).
template <bool FEW>
__device__ __forceinline__ int draw_row(const FwdParams& p, int home, int cut) {
  for (int from = home;;) {
    const int t = kResident + (int)atomicAdd(p.tickets + (size_t)from * p.ticket_stride, 1u);
    if (t < places_of<FEW>(p, from, cut)) {
      const int row = row_at_place<FEW>(p, from, t, cut);
      if (row >= 0) return row;
      continue;
    }
    int most = 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const uint32_t drawn =
          __hip_atomic_load(p.tickets + (size_t)x * p.ticket_stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int left = places_of<FEW>(p, x, cut) - kResident - (int)drawn;
      if (left > most) {
        most = left;
        from = x;
      }
    }
    if (most == 0) return -1;
  }
}

typedef const __attribute__((address_space(4))) FwdParams* const_params_ptr;
typedef const __attribute__((address_space(4))) FwdParams& ParamsRef;

// Step 0 of a call with few rows: nothing was skipped on entry, a row is one run (two, if its visit starts at a
// diagonal tile that is not the first), what the rows mark goes to newly_rows; the later steps' counters start at zero.
// The launch that cleared them before the kernel cost 1.5-3.4 us (one call of 2 rows x 1 tile 8.1 -> 6.7 us, 32 x 4
// 14.7 -> 12.5, 120 x 2 12.8 -> 9.4).  All the call's threads share it (by one workgroup's, counters of 16384 steps
// held up a call of 135 x 15 from 31.3 to 35.5 us); more than kClearWords for each of them are cleared by a launch
// beforehand all the same.
__device__ __forceinline__ void clear_counters(const FwdParams& p, int thread, int threads) {
  for (int64_t x = thread; x < p.stat_words; x += threads) {
    const int runs = p.rows_total + (p.diagonal_first ? p.rows_total - quotient(p.rows_total, p.Tq, p.per_Tq) : 0);
    p.stats_all[x] = x == 2 ? (unsigned long long)runs : 0ull;
  }
}

// Live tiles of mask word w as it stands.
__device__ __forceinline__ int live_in_word(uint64_t skipped, int w, int Tk) {
  const uint64_t tiles = Tk - 64 * w >= 64 ? ~0ull : (1ull << (Tk - 64 * w)) - 1ull;
  return __popcll(~skipped & tiles);
}
// Lane 0: the sum of what lanes 0 .. W-1 hold (the others hold 0).
__device__ __forceinline__ int sum_words(int n, int W) {
  for (int d = 1; d < W; d <<= 1) n += __shfl_xor(n, d, 64);
  return n;
}

// The end of a row without lists, by one wave: the tiles that fired (lane w: word w) join the Skip-Mask row as it was
// on entry (`skipped`; only of interest where something fired or live_next is set), the step's counter moves.
__device__ __forceinline__ void finish_mask_row(ParamsRef p, int row, int lane, uint64_t skipped, uint64_t fired) {
  if (lane < p.W && (p.fresh || fired)) p.bits[(size_t)row * p.W + lane] = skipped | fired;
  if (p.marked && fired) store_through(p.marked + p.table_calls, 1u);
  if (p.live_next) {
    const int n = sum_words(lane < p.W ? live_in_word(skipped | fired, lane, p.Tk) : 0, p.W);
    if (lane == 0) p.live_next[row] = (uint32_t)n;
  }
  if (!p.stat_newly) return;
  if (!p.fresh || !p.newly_rows) {
    if (fired) atomicAdd(p.stat_newly, (unsigned long long)__popcll(fired));
    return;
  }
  const int n = sum_words(__popcll(fired), p.W);
  if (lane == 0) p.newly_rows[row] = (uint32_t)n;
}

// Adds up the partial results of a row's pieces, in their order whichever arrived last, into what the end of the kernel
// expects of a whole row.  Loads have agent scope, like the stores (kStoreThrough); two pieces' are in flight together:
// 0.7 us a piece.
template <int QB, bool IMM>
__device__ __forceinline__ void merge_pieces(State<QB, IMM>& st, ParamsRef p, float c, int piece, int pieces, int wave,
                                             int lane) {
  const float* ps = p.seg_stat + (size_t)piece * 2 * kTile + 32 * wave + (lane & 31);
  auto stat = [&](int s, int which) {
    return __hip_atomic_load(ps + (s * 2 + which) * kTile, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  float m[kMaxPieces], l[kMaxPieces], top = kNoMax, sum = 0.f;
#pragma unroll
  for (int s = 0; s < kMaxPieces; ++s) {
    m[s] = stat(min(s, pieces - 1), 0);
    l[s] = stat(min(s, pieces - 1), 1);
    top = fmaxf(top, m[s]);
  }
  for (int s = kMaxPieces; !IMM && s < pieces; ++s) top = fmaxf(top, stat(s, 0));  // (rows cut alike)
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) st.oacc[0][db][r] = 0.f;
  auto add_two = [&](int s0, const float (&m)[2], const float (&l)[2]) __attribute__((always_inline)) {
    u32x4 x[2][16];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const auto po = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(p.seg_o + ((size_t)(piece + min(s0 + u, pieces - 1)) * 4 + wave) * 4096), 0, 4 * 4096, 0x00020000);
#pragma unroll
      for (int g = 0; g < 16; ++g) x[u][g] = __builtin_amdgcn_raw_buffer_load_b128(po, 16 * lane, 1024 * g, kStoreThrough);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (s0 + u >= pieces) break;
      const float f = __builtin_amdgcn_exp2f((m[u] - top) * c);
      sum += f * l[u];
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        const f32x4 v = __builtin_bit_cast(f32x4, x[u][g]);
#pragma unroll
        for (int r = 0; r < 4; ++r) st.oacc[0][g >> 2][4 * (g & 3) + r] += f * v[r];
      }
    }
  };
#pragma unroll
  for (int s0 = 0; s0 < kMaxPieces; s0 += 2) {
    if (s0 >= pieces) break;
    add_two(s0, {m[s0], m[s0 + 1]}, {l[s0], l[s0 + 1]});
  }
  for (int s0 = kMaxPieces; !IMM && s0 < pieces; s0 += 2) {
    const int s1 = min(s0 + 1, pieces - 1);
    add_two(s0, {stat(s0, 0), stat(s1, 0)}, {stat(s0, 1), stat(s1, 1)});
  }
  st.m_run[0] = top;
  st.l_run[0] = 0.5f * sum;  // (each half of the wave: half of the row sum)
}

// The tiles of piece `s` of a row that fire, by one wave: lane l holds Q rows 2l and 2l+1 and walks the row maxima that the
// pieces have left with the maximum carried over from the pieces before (see merge_segments_kernel).  Lane w returns word w.
template <class Pinned>
__device__ __forceinline__ uint64_t judge_piece(ParamsRef p, int row, int cut_row, int i, int piece, int pieces, int s,
                                                int lane, Pinned pinned) {
  uint64_t fired = 0;
  LiveWalk walk;
  int cnt, nruns;
  walk.open(LiveWalk::load(p.bits + (size_t)row * p.W, p.fresh, p.W), p.Tk, p.W, p.diagonal_first ? i : 0);
  walk.count(cnt, nruns);
  const auto mloc = __builtin_amdgcn_make_buffer_rsrc((void*)(p.seg_mloc + (size_t)cut_row * p.Tk * kTile), 0,
                                                      p.Tk * kTile * 4, 0x00020000);
  const auto stat = __builtin_amdgcn_make_buffer_rsrc((void*)(p.seg_stat + (size_t)piece * 2 * kTile), 0,
                                                      pieces * 2 * kTile * 4, 0x00020000);
  auto pair_of = [&](auto rsrc, int offset) {
    return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, 8 * lane, offset, kStoreThrough));
  };
  const bool valid0 = i * kTile + 2 * lane < p.N, valid1 = i * kTile + 2 * lane + 1 < p.N;
  f32x2 run = {-INFINITY, -INFINITY};
#pragma unroll
  for (int x = 0; x < kMaxPieces - 1; ++x) {
    const f32x2 m = pair_of(stat, min(x, pieces - 1) * 2 * kTile * 4);
    run[0] = x < s ? fmaxf(run[0], m[0]) : run[0];
    run[1] = x < s ? fmaxf(run[1], m[1]) : run[1];
  }
  for (int x = kMaxPieces - 1; x < s; ++x) {  // (rows cut alike)
    const f32x2 m = pair_of(stat, x * 2 * kTile * 4);
    run[0] = fmaxf(run[0], m[0]);
    run[1] = fmaxf(run[1], m[1]);
  }
  const int t0 = segment_start(cnt, s, pieces), t1 = segment_start(cnt, s + 1, pieces);
  if (t0 == t1) return fired;
  walk.rewind();
  walk.skip(t0);
  constexpr int kAhead = 8;  // tiles whose loads are in flight together
  for (int t = t0; t < t1; t += kAhead) {
    int j[kAhead];
    f32x2 m[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      j[u] = u > 0 ? j[u - 1] : 0;
      walk.next(j[u]);
      m[u] = pair_of(mloc, j[u] * kTile * 4);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (t + u >= t1) break;
      run[0] = fmaxf(run[0], m[u][0]);
      run[1] = fmaxf(run[1], m[u][1]);
      const bool ok = (!valid0 || (m[u][0] - run[0]) * p.scale <= p.thr) &&
                      (!valid1 || (m[u][1] - run[1]) * p.scale <= p.thr);
      if (__all(ok) && !pinned(j[u]) && lane == (j[u] >> 6)) fired |= 1ull << (j[u] & 63);
    }
  }
  return fired;
}

// x plus that of all lower lanes; the largest x >= 0 of the wave.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8: within 16 lanes
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15, 31
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return x;
}
__device__ __forceinline__ int wave_max(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

// Few rows that a mask has made unequal: every row is cut into ceil(live tiles / g) pieces, one workgroup each, with
// the smallest g (found from below) for which the workgroups that run side by side do; the piece that this workgroup
// computes.  All workgroups have to find the same cut, so the rows' live tiles come from counts made before this launch
// and not from the mask, which rows that end early change while workgroups of a busy chip may still have to start.
// (Each row's own tiles do come from the mask, and nobody changes them before all of its pieces have arrived: any
// counts give right results.)  Literal PV skip: only rows of protected tokens, whose tiles need no verdict, are cut.
// Where the counts say that the mask is empty, the rows are cut alike, as where the caller knows that it is: what a
// call gives depends on the mask, not on how it came about.  They are also cut alike, in as many rounds of workgroups
// as it takes, where one round would leave most rows nearly whole: us, 40 % of the tiles of each row skipped, 15 % in
// brackets, one round -> alike: 348 x 87 205 -> 192, 300 x 60 (175 -> 153), 304 x 304 597 -> 493, 150 x 150 165 -> 147,
// 129 x 129 (191 -> 171).
struct Piece {
  int row, index, pieces, first;  // (row -1: no piece, kAlike: cut alike; first: number of the row's first piece)
};
constexpr int kAlike = -2;
template <bool IMM>
__device__ __forceinline__ Piece pick_piece(const FwdParams& p, int xcd, int slot, int lane) {
  const int rows = p.rows_total;
  constexpr int kPerLane = kFewRows / 64;
  const int per_lane = (rows + 63) / 64;
  // every wave for itself, all loads in flight together (through LDS, one wave for all, the pieces were found 0.6 us later)
  const auto live = __builtin_amdgcn_make_buffer_rsrc((void*)p.live_rows, 0, rows * 4, 0x00020000);
  int c[kPerLane], tiles = 0, longest = 0;
#pragma unroll
  for (int k = 0; k < kPerLane; ++k)
    c[k] = k < per_lane ? (int)__builtin_amdgcn_raw_buffer_load_b32(live, 4 * (lane * per_lane + k), 0, 0) : 0;
  bool alike = true;
#pragma unroll
  for (int k = 0; k < kPerLane; ++k) {
    const int r = lane * per_lane + k;
    const bool is_row = k < per_lane && r < rows;
    alike = alike && (!is_row || c[k] == p.Tk);
    if constexpr (IMM) {
      const int i = r - (int)__umulhi((uint32_t)r, p.per_Tq) * p.Tq, at = i < p.Tq ? i : i - p.Tq;
      if (!(at * kTile < p.protect_start + p.protect_len && p.protect_start < (at + 1) * kTile)) c[k] = 1;
    }
    c[k] = is_row ? max(c[k], 1) : -(1 << 20);  // (no row: no piece, whatever g)
    tiles += max(c[k], 0);
    longest = max(longest, c[k]);
  }
  if (__all(alike)) return {kAlike, 0, 1, 0};
  tiles = __builtin_amdgcn_readlane(wave_scan(tiles), 63);
  longest = wave_max(longest);
  int g = max(quotient(tiles + p.piece_units - 1, p.piece_units), quotient(longest + kMaxPieces - 1, kMaxPieces));
  int n[kPerLane], mine, upto, total;
  for (;;) {
    const float inv = __builtin_amdgcn_rcpf((float)g), add = ((float)g - 0.5f) * inv;
    mine = 0;
#pragma unroll
    for (int k = 0; k < kPerLane; ++k) {  // ceil(c / g): (c + g - 1 + 1/2) / g is never near an integer
      n[k] = 0;
      if (k < per_lane) n[k] = max((int)__builtin_fmaf((float)c[k], inv, add), 0);
      mine += n[k];
    }
    upto = wave_scan(mine);
    total = __builtin_amdgcn_readlane(upto, 63);
    if (total <= p.piece_units || g >= longest) break;  // (g = longest: a piece for every row, and rows <= units)
    g = max(g + 1, quotient(g * total, p.piece_units));
    if (4 * g > 3 * longest) g = longest;  // not worth the merging
  }
  if constexpr (!IMM) {  // (a piece costs about two tiles' time besides its own)
    const int rounds = quotient(rows * p.equal_pieces + p.piece_units - 1, p.piece_units);
    const int each = quotient(longest + p.equal_pieces - 1, p.equal_pieces);
    if (p.equal_pieces > 1 && g > rounds * (each + 2)) return {kAlike, 0, 1, 0};
  }
  Piece out = {-1, 0, 1, 0};
  const int share = (total + 7) / 8, unit = xcd * share + slot;
  if (slot >= share || unit >= total) return out;
  const int owner = __popcll(__ballot(upto <= unit));  // lane that holds the row
  int first = __builtin_amdgcn_readlane(upto - mine, owner);
#pragma unroll
  for (int k = 0; k < kPerLane; ++k) {
    const int nk = __builtin_amdgcn_readlane(n[k], owner);
    if (out.row < 0 && unit < first + nk) out = {owner * per_lane + k, unit - first, nk, first};
    first += nk;
  }
  return out;
}

template <int QB, bool IMM, bool FEW, bool PAIR>
__global__ __launch_bounds__(Geo<QB>::kThreads * (PAIR ? 2 : 1), 2 / QB) void lite_attn_fwd_kernel(const FwdParams p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  static_assert(!PAIR || (FEW && QB == 1), "two groups of four waves: only with few rows");
  constexpr int kWaves = Geo<QB>::kWaves, kChunks = Geo<QB>::kChunks;
  constexpr int kThreads = Geo<QB>::kThreads * (PAIR ? 2 : 1);
  if constexpr (FEW) touch_arguments(sizeof(FwdParams));
  const int tid = threadIdx.x, lane = tid & 63, wave = (tid >> 6) & (kWaves - 1);
  const int grp = PAIR ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0;  // PAIR: which half of every tile's columns
  const int lq = lane & 31;

  // Consecutive workgroup ids land on different XCDs (id % 8): workgroup `slot` of an XCD computes the row at that
  // place of the XCD's list in the schedule table (deal_rows(): chunks of kChunkRows rows of one head side by
  // side, so that the workgroups sharing one L2 stream the same K/V; equal work per XCD; long rows first) or, after the
  // first round, the one that it draws (draw_row). FEW: the table of schedule_rows_kernel if the call has one; else the
  // (head, segment, row) triples, numbered row-fastest, an eighth to every XCD, so that the rows walking the same K/V
  // tiles of a head share an L2; beyond kSchedRows rows, where the XCDs' shares would be whole heads, chunks of rows
  // dealt to the XCDs in turn.  Over 200 seeded sets of head densities (260-1000 heads, alike to 0.05 against 0.95,
  // with and without a period) the busiest XCD has 1.035 times the mean work, at worst 1.18; eighths give 4.4 where an
  // eighth of the heads is dense and the others 10 % live.  320 heads x 128 tiles, ms: that mask 30.6 -> 9.3, half the
  // heads 90 % and half 15 % live 34.8 -> 21.7, all 45 % 19.6 both ways (chunks of 32 rows 19.7, of 128 19.6).
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int row = -1, i, bh, seg = 0;
  int pieces = 1, piece = 0;  // a row cut into pieces (pick_piece): how many, and the first one's partial result
  if (FEW && !p.tickets && p.piece_units && !p.alike) {
    const Piece mine = pick_piece<IMM>(p, xcd, slot, lane);
    if (mine.row == -1) return;
    row = mine.row;
    seg = mine.index;
    pieces = mine.pieces;
    piece = mine.first;
  }
  if (FEW && !p.tickets) {
    if (row < 0) {  // all rows alike: segments, or as many pieces
      const int n = IMM ? 1 : p.parts, units = p.rows_total * n, share = (units + 7) / 8;
      const int unit = xcd * share + slot;
      if (slot >= share || unit >= units) return;
      const int u = quotient(unit, p.Tq, p.per_Tq);
      bh = n == 1 ? u : quotient(u, n, p.per_parts);
      seg = u - bh * n;
      i = unit - u * p.Tq;
      row = bh * p.Tq + i;
      if constexpr (!IMM) {
        pieces = p.equal_pieces;
        piece = row * pieces;
      }
    } else {
      bh = quotient(row, p.Tq, p.per_Tq);
      i = row - bh * p.Tq;
    }
  } else {
    int cut = 0;  // rows of each eighth that are cut
    if (FEW && p.cut_rows > 0) {
      cut = !p.scheduled || p.slots[(size_t)(xcd + 1) * p.per_xcd - kTableTail] ? p.cut_rows : 0;
      // (a table made by an earlier call, for an empty mask: whether any call since has marked a tile)
      for (int x = 0; cut > 0 && x < p.table_calls; ++x)
        if (p.marked[x]) cut = 0;
    }
    if (slot < p.resident) row = row_at_place<FEW>(p, xcd, slot, cut);
    if (row < 0) {
      if (p.resident == kNoDraws) return;
      int* told = reinterpret_cast<int*>(smem + (PAIR ? kPairFlagsOff : kFlagsOff));
      if (tid == 0) *told = draw_row<FEW>(p, xcd, cut);
      __syncthreads();
      row = __builtin_amdgcn_readfirstlane(*told);
      if (row < 0) return;
      __syncthreads();  // (the flags are this word's next user)
    }
    if constexpr (FEW) {
      seg = row >> kPieceShift;
      row &= (1 << kPieceShift) - 1;
      if (cut > 0) {
        const int share = (p.rows_total + 7) / 8, x = quotient(row, share), r = row - x * share - (share - cut);
        if (r >= 0) {
          pieces = p.cut_pieces;
          piece = (x * cut + r) * pieces;
        }
      }
    }
    bh = quotient(row, p.Tq, p.per_Tq);
    i = row - bh * p.Tq;
  }
  const int b = quotient(bh, p.H, p.per_H);
  const int64_t base = (int64_t)b * p.stride_b + (int64_t)(bh - b * p.H) * p.stride_h;
  uint16_t* ob = p.out + base;
  const int N = p.N;
  const bool split = FEW && (p.nseg > 1 || pieces > 1);
  const int part = piece << 8 | pieces << 4 | seg;  // (one scalar register across the main loop)
  Lane<QB> ln;
  State<QB, IMM> st;
  ln.hi = lane >> 5;
  const uint32_t head_bytes = (uint32_t)(((int64_t)(N - 1) * p.stride_n + 128) * 2);
  auto load_q = [&]() {  // Q^T fragments: B operand of S^T = K Q^T, kept for the whole row
    const auto qr = __builtin_amdgcn_make_buffer_rsrc((void*)(p.q + base), 0, head_bytes, 0x00020000);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int qrow = i * kTile + 32 * (QB * wave + qb) + lq;
      ln.qvalid[qb] = qrow < N;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        if constexpr (FEW) {  // rows past the end of the sequence read as zeros: no branch per load
          st.qf[qb][kk] = __builtin_bit_cast(
              bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                          qr, (int)((uint32_t)qrow * (uint32_t)(p.stride_n * 2) + 16 * ln.hi), 32 * kk, 0));
        } else {
          uint4 raw = {0u, 0u, 0u, 0u};
          if (ln.qvalid[qb])
            raw = *reinterpret_cast<const uint4*>(p.q + base + (int64_t)qrow * p.stride_n + 16 * kk + 8 * ln.hi);
          st.qf[qb][kk] = *reinterpret_cast<bf16x8*>(&raw);
        }
      }
    }
  };
  char* const stages = smem + (PAIR ? grp * 4 * kStageBytes : 0);  // this group's stage buffers
  auto lane_constants = [&]() {
    ln.N = N;
    ln.scale = p.scale;
    ln.thr = p.thr;
    ln.c = p.scale * 1.4426950408889634f;
    ln.stride2 = (uint32_t)(p.stride_n * 2);
    ln.krsrc = make_rsrc(p.k + base, head_bytes);
    const uint32_t vt_row_bytes = (uint32_t)p.Tk * kTile * 2;  // one feature row of V^T: n_pad bf16
    ln.vrsrc = FEW ? make_rsrc(p.v + base, head_bytes)
                   : make_rsrc(p.vt + (size_t)bh * 128 * ((size_t)p.Tk * kTile), 128u * vt_row_bytes);
    ln.lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(LA_LDS char*)stages + 1024 * kChunks * wave);
    ln.col = grp * kSub;
#pragma unroll
    for (int x = 0; x < kChunks; ++x) {
      const int r = 4 * (kChunks * wave + x) + (lane >> 4);  // row inside the stage that this lane's piece belongs to
      const int pc = lane & 15;                              // physical 16-byte chunk inside the 256-byte LDS row
      ln.kdma[x] = (uint32_t)r * ln.stride2 + 16 * (pc ^ (r & 15));
      if constexpr (FEW) {  // V stage: 64 token rows x 256 bytes; four rows' 64-byte pieces of a d-block meet all banks
        ln.vdma[x] = (uint32_t)r * ln.stride2 + 16 * (pc ^ (4 * (r & 3)));
        continue;
      }
      // V^T stage: 128 feature rows x 128 bytes; this lane's piece is row rv, physical 16-byte slot pv
      const int rv = 8 * (kChunks * wave + x) + (lane >> 3), pv = lane & 7;
      ln.vdma[x] = (uint32_t)rv * vt_row_bytes + 16 * (pv ^ ((rv >> 1) & 7));
    }
    const uint32_t lds0 = (uint32_t)(size_t)(LA_LDS char*)stages;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) ln.kread[kk] = lds0 + lq * 256 + ((32 * kk) ^ (16 * (ln.hi ^ (lq & 15))));
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      if constexpr (FEW) {  // d-block cc: row 4*hi + (lane>>2 & 3) of a chunk, 8-byte piece lane & 3 of its 16 features
        const int r = 4 * ln.hi + ((lane >> 2) & 3), c = 4 * cc + 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
        ln.vread[cc] = lds0 + r * 256 + 16 * (c ^ (4 * (r & 3))) + 8 * (lane & 1);
      } else {
        ln.vread[cc] = lds0 + lq * 128 + ((32 * cc + 16 * ln.hi) ^ (16 * ((lq >> 1) & 7)));
      }
    }
  };
  auto clear_odd_v = [&]() {  // the odd V^T buffer is read (times P~ = 0) before it is first filled: make it finite
#pragma unroll
    for (int x = tid & (64 * kWaves - 1); x < kStageBytes / 16; x += 64 * kWaves)
      *reinterpret_cast<uint4*>(stages + kVOff + kStageBytes + 16 * x) = uint4{0u, 0u, 0u, 0u};
  };
  LiveWalk walk;
  int cnt, nruns, t_lo = 0, t_hi;
  if constexpr (FEW) {
    // the mask row first, then Q, all in flight together.  With the arguments brought in at once and the divisions in
    // a few instructions: tiny layer's step 20.1 -> 19.3 us, options clip's 60.6 -> 59.1 (loading a word of K and V here
    // too, to have their pages mapped early, was slower: 20.3)
    const uint64_t skipped = LiveWalk::load(p.bits + (size_t)row * p.W, p.fresh, p.W);
    load_q();
    // what the main loop needs besides, while the mask row is on its way, and held here (the compiler would move it behind
    // the wait): 32 rows x 16 tiles, four steps, 66 -> 63 us, 72 x 12, three, 58.9 -> 56.7
    lane_constants();
    if (!IMM) clear_odd_v();
#pragma unroll
    for (int x = 0; x < kChunks; ++x) asm volatile("" : "+v"(ln.kdma[x]), "+v"(ln.vdma[x]));
#pragma unroll
    for (int x = 0; x < 4; ++x) asm volatile("" : "+v"(ln.kread[2 * x]), "+v"(ln.kread[2 * x + 1]), "+v"(ln.vread[x]));
    __builtin_amdgcn_sched_barrier(0);
    if (p.fresh) {  // no wait for the mask row
      walk.open(0, p.Tk, p.W, p.diagonal_first ? i : 0);
      asm volatile("" : "+v"(walk.lo), "+v"(walk.hi));
    } else {
      walk.open(skipped, p.Tk, p.W, p.diagonal_first ? i : 0);
    }
    walk.count(cnt, nruns);
    t_lo = segment_start(cnt, seg, p.nseg * pieces);
    t_hi = segment_start(cnt, seg + 1, p.nseg * pieces);
    if (p.fresh && p.newly_rows) {
      const int n = IMM ? 1 : p.parts;
      clear_counters(p, (row * n + seg) * kThreads + tid, p.rows_total * n * kThreads);
    }
  } else {
    cnt = (int)p.live_cnt[row];
    nruns = (int)p.nruns[row];
    t_hi = cnt;
  }
  // the Skip-List is read-only here: constant address space makes these wave-uniform reads scalar loads
  typedef const __attribute__((address_space(4))) uint32_t* const_u32_ptr;
  const_u32_ptr runs = (const_u32_ptr)(p.runs + (size_t)row * p.run_stride);
  int* flags = reinterpret_cast<int*>(smem + (PAIR ? kPairFlagsOff : kFlagsOff));
  float* xch = reinterpret_cast<float*>(smem + kPairXchOff);  // PAIR: group 1's row maxima, by parity of the tile
  // mask bits set by this workgroup during the call (thread 0 writes them, wave 0 reads them in the epilogue)
  uint64_t* fired_bits = reinterpret_cast<uint64_t*>(smem + kFiredOff);
  if (!FEW && p.build_next)
    for (int w = tid; w < p.W; w += kThreads) fired_bits[w] = 0;
  // statistics of the step: tiles skipped on entry, Skip-List entries
  if (tid == 0 && !(FEW && p.nseg > 1) && seg == 0 && p.stat_newly && !(FEW && p.fresh && p.newly_rows)) {
    atomicAdd(p.stat_skipped_in, (unsigned long long)(p.Tk - cnt));
    atomicAdd(p.stat_runs, (unsigned long long)nruns);
  }

  if constexpr (!FEW) lane_constants();
  const bool q_pinned = p.protect_len > 0 && i * kTile < p.protect_start + p.protect_len &&
                        p.protect_start < min(N, (i + 1) * kTile);

  // whether tile (i, j) meets the pinned token range; FEW: asked only of tiles that would fire, with the kernel arguments
  // read again (scalar registers are short in the main loop)
  auto pinned = [&](int j) -> bool {
    const_params_ptr a = (const_params_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    const int lo = a->protect_start, hi = lo + a->protect_len, n = a->N;
    return hi > lo && ((i * kTile < hi && lo < min(n, (i + 1) * kTile)) || (j * kTile < hi && lo < min(n, (j + 1) * kTile)));
  };

  if constexpr (!FEW) load_q();
  st.grew_prev = false;
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    st.l_pend[qb][0] = st.l_pend[qb][1] = 0.f;
    st.alpha_prev[qb] = 1.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.oacc[qb][db][r] = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) st.pw[qb][e] = 0u;
    st.m_run[qb] = kNoMax;     // running row max of the raw dot products (m_{i,j-1} * sqrt(d))
    st.l_run[qb] = 0.f;        // this lane's half of the row sum
    st.mloc_tile[qb] = -INFINITY;
  }
  st.mloc_prev = st.m_all = -INFINITY;
  unsigned newly = 0;

  // lane 0 writes the wave's predicate flag, every other lane a private dummy word (keeps the stage branch-free)
  int* flag_slot0 = lane == 0 ? flags + wave : flags + 8 + lane;
  int* flag_slot1 = lane == 0 ? flags + 4 + wave : flags + 8 + lane;

  // FEW: lane w of wave 0 collects the bits of mask word w that this call sets
  uint64_t fired_word = 0;
  if (t_hi > t_lo) {
    // Walk the run-length Skip-List with a cursor kept two tiles ahead of the tile being computed, so that the
    // scalar load of the next run entry is off the critical path.  At the end of the list the cursor stays put.
    int c_run = 0, c_j = 0, c_end = 0;
    if constexpr (FEW) {
      walk.skip(t_lo);
      walk.next(c_j);
    } else {
      const uint32_t e = runs[0];
      c_j = (int)(e & 0xffffu);
      c_end = (int)(e >> 16);
    }
    auto advance = [&]() {
      if constexpr (FEW) {
        // behind the last tile, one before the sequence: past the end of the buffer, so that no K is fetched that nobody
        // needs (0.3-0.9 % of calls with few tiles a workgroup)
        if (!walk.next(c_j)) c_j = -1;
      } else if (c_j + 1 < c_end) {
        ++c_j;
      } else if (c_run + 1 < nruns) {
        ++c_run;
        const uint32_t e = runs[c_run];
        c_j = (int)(e & 0xffffu);
        c_end = (int)(e >> 16);
      }
    };
    int j_cur = c_j;
    advance();
    int j_nxt = c_j;
    // the last tile of a sequence that ends inside it needs its columns masked; the stages compare their tile index
    // with this one on the scalar unit (a bool would travel between their blocks as a lane mask)
    const int j_tail = (N & (kTile - 1)) != 0 ? p.Tk - 1 : -1;

    // prologue: K of stages 0 and 1; then S^T(0)
    if (!FEW && !IMM) clear_odd_v();
    dma_stage<QB, kKOff>(ln.krsrc, ln.kdma, (uint32_t)(j_cur * kTile + ln.col) * ln.stride2, ln.lds_wave);
    dma_stage<QB, kKOff + kStageBytes>(
        ln.krsrc, ln.kdma, (uint32_t)(PAIR ? j_nxt * kTile + ln.col : j_cur * kTile + kSub) * ln.stride2, ln.lds_wave);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    mma_qk<QB>(st.sA, st.qf, kKOff, ln.kread);
    __syncthreads();

    // IMM: every wave reads the four per-wave results and the pinned-range rule itself (it needs the verdict to
    // gate the tile's PV products); returns whether the tile fired (wave-uniform)
    auto finish_tile_imm = [&](int t, int j) -> bool {
      const int4 f = *reinterpret_cast<const int4*>(flags + (t & 1) * 4);
      static_assert(!IMM || kWaves == 4, "four per-wave flags per tile");
      const int all = __builtin_amdgcn_readfirstlane(f.x & f.y & f.z & f.w);
      bool fired;
      if constexpr (FEW) {
        fired = all && !pinned(j);
      } else {
        const bool k_pinned = p.protect_len > 0 && j * kTile < p.protect_start + p.protect_len &&
                              p.protect_start < min(N, (j + 1) * kTile);
        fired = all && !q_pinned && !k_pinned;
      }
      if constexpr (FEW) {
        if (fired && tid == (j >> 6)) fired_word |= 1ull << (j & 63);
      } else if (tid == 0 && fired) {
        atomicOr(reinterpret_cast<unsigned long long*>(p.bits + (size_t)row * p.W + (j >> 6)), 1ull << (j & 63));
        fired_bits[j >> 6] |= 1ull << (j & 63);
        ++newly;
      }
      return fired;
    };
    // Deferred marking: the per-wave results of a finished tile meet in LDS; wave 0 combines them and updates the
    // mask, not at the barrier that ends the tile (it would be late for the next stage by the latency of an LDS read,
    // and the other three waves would wait for it at the next barrier) but during the first stage of the next tile.
    const bool wave0 = __builtin_amdgcn_readfirstlane(tid >> 6) == 0;
    int4 vflags = {0, 0, 0, 0};
    const int* v_slot = flags;  // LDS slot of the tile whose verdict is pending
    int v_j = -1;               // its K/V tile index (-1: none pending)
    auto mark_if_fired = [&](int all, int j) {
      if constexpr (FEW) {
        if (__builtin_amdgcn_readfirstlane(all) && !pinned(j) && tid == (j >> 6)) fired_word |= 1ull << (j & 63);
      } else if (tid == 0 && all) {
        const bool k_pinned = p.protect_len > 0 && j * kTile < p.protect_start + p.protect_len &&
                              p.protect_start < min(N, (j + 1) * kTile);
        if (!q_pinned && !k_pinned) {
          atomicOr(reinterpret_cast<unsigned long long*>(p.bits + (size_t)row * p.W + (j >> 6)), 1ull << (j & 63));
          fired_bits[j >> 6] |= 1ull << (j & 63);
          ++newly;
        }
      }
    };
    // split rows: whether a tile fires depends on the segments before this one; its row maxima go to the merge pass
    float* mloc_out = nullptr;
    if constexpr (FEW) {
      const int at = p.tickets ? quotient(part >> 8, part >> 4 & 15) : row;  // (beyond kFewRows: by cut row)
      mloc_out = p.seg_mloc + (size_t)at * p.Tk * kTile + 32 * wave + lq;
    }
    auto verdict_load = [&]() {
      static_assert(IMM || kWaves == 4, "four per-wave flags per tile");
      if (split) {
        if (v_j >= 0 && ln.hi == 0 && ln.thr > -INFINITY) store_through(mloc_out + v_j * kTile, st.mloc_tile[0]);
        return;
      }
      if (wave0) vflags = *reinterpret_cast<const int4*>(v_slot);
    };
    auto verdict_commit = [&]() {
      if (!split && wave0 && v_j >= 0) mark_if_fired(vflags.x & vflags.y & vflags.z & vflags.w, v_j);
    };
    bool pv_on = false;  // IMM: the previous tile did not fire, its PV products are due
    int j_prev = j_cur;
    if constexpr (PAIR) {
      // One stage per tile.  Tile t's verdict: group 1's row maxima reach LDS at the end of stage t; during stage t+1
      // group 0 joins them with its own, judges the tile and puts the four per-wave results into the flags (split
      // rows: stores the joint maxima for the merge pass instead); during stage t+2 wave 0 updates the mask (IMM: all
      // waves read the verdict before stage t+2, which holds the tile's PV product).
      int j_pp = -1;  // the tile before the previous one
      j_prev = -1;
      float other = 0.f;
      auto join = [&](int parity) {  // group 0: the previous tile's maxima over all columns, and its judgement
        if (grp != 0) return;
        const float mloc = fmaxf(st.mloc_prev, other);
        st.m_all = fmaxf(st.m_all, mloc);
        if (split && !IMM) {
          if (ln.hi == 0 && ln.thr > -INFINITY) store_through(mloc_out + j_prev * kTile, mloc);
        } else {
          const bool ok = __all(!ln.qvalid[0] || (mloc - st.m_all) * ln.scale <= ln.thr);
          *(lane == 0 ? flags + 4 * parity + wave : flags + 8 + lane) = ok ? 1 : 0;
        }
      };
      auto imm_verdict = [&](int parity, float pend) {  // of tile j_pp: marks it, or adds its row sums
        pv_on = false;
        if (j_pp < 0) return;
        const int4 f = *reinterpret_cast<const int4*>(flags + 4 * parity);
        const int all = __builtin_amdgcn_readfirstlane(f.x & f.y & f.z & f.w);
        pv_on = !(all && !pinned(j_pp));
        if (pv_on)
          st.l_run[0] += pend;
        else if (tid == (j_pp >> 6))
          fired_word |= 1ull << (j_pp & 63);
      };
      auto one = [&](auto par) __attribute__((always_inline)) {
        constexpr int H = decltype(par)::value;
        advance();
        const int j_nn = c_j;
        if constexpr (IMM) imm_verdict(H, st.l_pend[0][H]);
        auto load = [&]() {
          if (grp == 0 && j_prev >= 0) other = xch[(H ^ 1) * kTile + 32 * wave + lq];
          if (!IMM && !split && wave0) vflags = *reinterpret_cast<const int4*>(flags + 4 * H);
        };
        auto commit = [&]() {
          if (j_prev >= 0) join(H ^ 1);
          if (!IMM && !split && wave0 && j_pp >= 0) mark_if_fired(vflags.x & vflags.y & vflags.z & vflags.w, j_pp);
        };
        auto end = [&](float mx) {
          st.mloc_prev = mx;
          if (grp == 1 && ln.hi == 0) xch[H * kTile + 32 * wave + lq] = mx;
        };
        stage<QB, H, IMM, true, true>(st, ln, smem, j_cur, j_nn, flags, j_tail, max(j_prev, 0), !IMM || pv_on, load,
                                      commit, end);
        j_pp = j_prev;
        j_prev = j_cur;
        j_cur = j_nxt;
        j_nxt = j_nn;
      };
      int last = 0;  // parity of the last tile
      for (int t = t_lo;;) {
        last = 0;
        one(std::integral_constant<int, 0>{});
        if (++t >= t_hi) break;
        last = 1;
        one(std::integral_constant<int, 1>{});
        if (++t >= t_hi) break;
      }
      // drain: the last tile's PV product (IMM: the last two tiles'), its verdict and that of the tile before it
      if (IMM)
        dma_stage<QB, kVOff>(ln.vrsrc, ln.vdma, (uint32_t)(j_prev * kTile + ln.col) * ln.stride2,
                             ln.lds_wave + (uint32_t)last * kStageBytes);
      if (grp == 0) other = xch[last * kTile + 32 * wave + lq];
      if constexpr (IMM) {
        imm_verdict(last ^ 1, last ? st.l_pend[0][0] : st.l_pend[0][1]);
      } else if (!split && wave0 && j_pp >= 0) {
        vflags = *reinterpret_cast<const int4*>(flags + 4 * (last ^ 1));
        mark_if_fired(vflags.x & vflags.y & vflags.z & vflags.w, j_pp);
      }
      join(last);
      if (!IMM) mma_pv<QB, true>(st.oacc, st.pw, kVOff + last * kStageBytes, ln.vread);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      j_pp = j_prev;
      if constexpr (IMM) {
        auto drain = [&](const uint32_t (&p_prev)[QB][16], const uint32_t (&p_last)[QB][16]) {
          if (pv_on) mma_pv<QB, true>(st.oacc, p_prev, kVOff + (last ^ 1) * kStageBytes, ln.vread);
          if (st.grew_prev) {
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
              for (int r = 0; r < 16; ++r) st.oacc[0][db][r] *= st.alpha_prev[0];
          }
          imm_verdict(last, last ? st.l_pend[0][1] : st.l_pend[0][0]);
          if (pv_on) mma_pv<QB, true>(st.oacc, p_last, kVOff + last * kStageBytes, ln.vread);
        };
        if (last)
          drain(st.pw0, st.pw);
        else
          drain(st.pw, st.pw0);
      } else if (!split && wave0) {
        vflags = *reinterpret_cast<const int4*>(flags + 4 * last);
        mark_if_fired(vflags.x & vflags.y & vflags.z & vflags.w, j_prev);
      }
      __syncthreads();
      // group 1's share joins group 0's: accumulators as the lanes hold them, through group 1's stage buffers
      float4* hand = reinterpret_cast<float4*>(smem + 4 * kStageBytes) + (size_t)wave * 1024 + lane;
      float* hand_stat = xch;  // [row maximum, row sum][128]
      const float l_half = other_half_sum(st.l_run[0]);
      if (grp == 1) {
#pragma unroll
        for (int g = 0; g < 16; ++g) {
          const f32x16& a = st.oacc[0][g >> 2];
          const int r = 4 * (g & 3);
          hand[64 * g] = float4{a[r], a[r + 1], a[r + 2], a[r + 3]};
        }
        if (ln.hi == 0) {
          hand_stat[32 * wave + lq] = st.m_run[0];
          hand_stat[kTile + 32 * wave + lq] = l_half;
        }
      }
      __syncthreads();
      if (grp == 0) {
        const float m1 = hand_stat[32 * wave + lq], l1 = hand_stat[kTile + 32 * wave + lq];
        const float top = fmaxf(st.m_run[0], m1);
        const float f0 = __builtin_amdgcn_exp2f((st.m_run[0] - top) * ln.c), f1 = __builtin_amdgcn_exp2f((m1 - top) * ln.c);
        st.m_run[0] = top;
        st.l_run[0] = 0.5f * (f0 * l_half + f1 * l1);  // (each half of the wave: half of the row sum)
#pragma unroll
        for (int g = 0; g < 16; ++g) {
          f32x16& a = st.oacc[0][g >> 2];
          const int r = 4 * (g & 3);
          const float4 b = hand[64 * g];
          a[r] = f0 * a[r] + f1 * b.x;
          a[r + 1] = f0 * a[r + 1] + f1 * b.y;
          a[r + 2] = f0 * a[r + 2] + f1 * b.z;
          a[r + 3] = f0 * a[r + 3] + f1 * b.w;
        }
      }
    }
    for (int t = t_lo; !PAIR && t < t_hi; ++t) {
      advance();
      const int j_nn = c_j;  // needed one tile from now
      int* fs = (t & 1) ? flag_slot1 : flag_slot0;
      if constexpr (PAIR) {
      } else if constexpr (IMM) {
        stage<QB, 0, true, FEW, false>(st, ln, smem, j_cur, j_nxt, fs, j_tail, j_prev, pv_on);
        stage<QB, 1, true, FEW, false>(st, ln, smem, j_cur, j_nxt, fs, j_tail, j_cur, pv_on);
        pv_on = !finish_tile_imm(t, j_cur);
        if (pv_on) {
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) st.l_run[qb] += st.l_pend[qb][0];
        }
        j_prev = j_cur;
      } else {
        stage<QB, 0, false, FEW, false>(st, ln, smem, j_cur, j_nxt, fs, j_tail, 0, true, verdict_load, verdict_commit);
        stage<QB, 1, false, FEW, false>(st, ln, smem, j_cur, j_nxt, fs, j_tail);
        v_slot = flags + (t & 1) * 4;
        v_j = j_cur;
      }
      j_cur = j_nxt;
      j_nxt = j_nn;
    }
    if constexpr (PAIR) {
    } else if constexpr (IMM) {
      // drain: the second V^T stage of the last tile is still to be loaded; then both of its PV products, the
      // rescale factor of its second stage in between
      dma_stage<QB, kVOff + kStageBytes>(ln.vrsrc, ln.vdma,
                                         (uint32_t)(j_prev * kTile + kSub) * (FEW ? ln.stride2 : 2u), ln.lds_wave);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (pv_on) mma_pv<QB, FEW>(st.oacc, st.pw0, kVOff, ln.vread);
      if (st.grew_prev) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
          for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.oacc[qb][db][r] *= st.alpha_prev[qb];
      }
      if (pv_on) mma_pv<QB, FEW>(st.oacc, st.pw, kVOff + kStageBytes, ln.vread);
    } else {
      // drain: O^T += V^T P~^T of the last stage (odd parity buffer), and the verdict on the last tile
      mma_pv<QB, FEW>(st.oacc, st.pw, kVOff + kStageBytes, ln.vread);
      verdict_load();
      verdict_commit();
    }
    __syncthreads();
  }
  // (the kernel arguments used from here on are read again from the argument segment instead of being kept in scalar
  // registers across the main loop)
  const_params_ptr e = (const_params_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(e));
  uint64_t skipped_on_entry = 0;
  if constexpr (FEW) {
    static_assert(QB == 1, "one Q block per wave");
    // partial result of a segment or piece: O^T accumulators as the lanes hold them (1 KB per store), the row maxima
    // (reference of the exponentials) and the row sums
    auto leave_partial = [&](size_t s, bool empty) {
      const auto po = __builtin_amdgcn_make_buffer_rsrc((void*)(e->seg_o + (s * 4 + wave) * 4096), 0, 4 * 4096, 0x00020000);
      if (!empty)
#pragma unroll
        for (int g = 0; g < 16; ++g) {
          const f32x16& a = st.oacc[0][g >> 2];
          const int r = 4 * (g & 3);
          const f32x4 o = {a[r], a[r + 1], a[r + 2], a[r + 3]};
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), po, 16 * lane, 1024 * g, kStoreThrough);
        }
      const float l = other_half_sum(st.l_run[0]);
      if (ln.hi == 0) {
        float* ps = e->seg_stat + s * 2 * kTile + 32 * wave + lq;
        store_through(ps, st.m_run[0]);
        store_through(ps + kTile, l);
      }
    };
    if (e->nseg > 1) {  // merged by a pass of its own
      if (grp == 0) leave_partial((size_t)row * e->nseg + (part & 15), t_hi == t_lo);
      return;
    }
    const int n_pieces = part >> 4 & 15, first_piece = part >> 8;
    if (n_pieces > 1) {  // merged by the piece that arrives last
      if (grp == 0) leave_partial((size_t)(first_piece + (part & 15)), false);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the partials are past the L2 before the arrival is)
      __syncthreads();
      int cut_row = row, counter = row;
      if (e->tickets) {
        cut_row = quotient(first_piece, n_pieces);
        const int x = quotient(cut_row, e->cut_rows);
        counter = x * e->arrive_stride + cut_row - x * e->cut_rows;
      }
      if (tid == 0) *flags = (int)atomicInc(e->arrive + counter, (unsigned)n_pieces - 1);
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(*flags) != n_pieces - 1) return;
      uint64_t(*fired)[64] = reinterpret_cast<uint64_t(*)[64]>(smem);
      if (grp == 0) merge_pieces<QB, IMM>(st, *e, ln.c, first_piece, n_pieces, wave, lane);
      if constexpr (!IMM) {
        if (ln.thr > -INFINITY) {
          if (grp == (PAIR ? 1 : 0)) {
            uint64_t f = 0;
            for (int s = wave; s < n_pieces; s += 4)
              f |= judge_piece(*e, row, cut_row, i, first_piece, n_pieces, s, lane, pinned);
            fired[wave][lane] = f;
          }
          __syncthreads();
          if (tid < 64) fired_word = fired[0][lane] | fired[1][lane] | fired[2][lane] | fired[3][lane];
          __syncthreads();  // (the results pass through the same memory)
        }
      }
    }
    skipped_on_entry = LiveWalk::load(e->bits + (size_t)row * e->W, e->fresh, e->W);
  } else {
    if (tid == 0 && newly && e->stat_newly) atomicAdd(e->stat_newly, (unsigned long long)newly);
  }

  // ---- epilogue: O = acc / l, transposed through LDS so that global stores are 16 B and row-contiguous ----
  char* sO = smem;
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    if (grp != 0) break;
    const float l = other_half_sum(st.l_run[qb]);
    const float inv = (l > 0.f) ? 1.f / l : 0.f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        uint2 w;
        w.x = pack_bf16x2(st.oacc[qb][db][4 * rg + 0] * inv, st.oacc[qb][db][4 * rg + 1] * inv);
        w.y = pack_bf16x2(st.oacc[qb][db][4 * rg + 2] * inv, st.oacc[qb][db][4 * rg + 3] * inv);
        *reinterpret_cast<uint2*>(sO + (32 * (QB * wave + qb) + lq) * kORow + 2 * (32 * db + 8 * rg + 4 * ln.hi)) = w;
      }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 2048 / kThreads; ++t) {
    const int r = (tid >> 4) + (kThreads / 16) * t;
    const int grow = i * kTile + r;
    const u32x4 o = *reinterpret_cast<const u32x4*>(sO + r * kORow + 16 * (tid & 15));
    if constexpr (FEW)  // (rows past the end of the sequence lie past the end of the buffer)
      __builtin_amdgcn_raw_buffer_store_b128(o, __builtin_amdgcn_make_buffer_rsrc((void*)ob, 0, head_bytes, 0x00020000),
                                             (int)((uint32_t)grow * ln.stride2 + 16 * (tid & 15)), 0, kStoreThrough);
    else if (grow < N)
      *reinterpret_cast<u32x4*>(ob + (int64_t)grow * p.stride_n + 8 * (tid & 15)) = o;
  }

  if constexpr (FEW) {  // behind the results, while these are on their way
    if (tid < 64) finish_mask_row(*e, row, lane, skipped_on_entry, fired_word);
    return;
  }
  // ---- second epilogue: the Skip-List this row will walk in the NEXT call, compacted from the mask row as this call
  // leaves it: the row as it was on entry (nobody else writes it) OR the bits this workgroup set, which it kept in
  // LDS, so that nothing depends on when its own atomics become visible to its loads.  The row's list is private to
  // this workgroup: it is overwritten in place, after its last read. ----
  if (e->build_next && wave == 0) {
    uint32_t ns, n;
    compact_row(e->bits + (size_t)row * e->W, [&](int w) { return fired_bits[w]; }, i, e->Tk, e->W, e->diagonal_first,
                e->runs + (size_t)row * e->run_stride, ns, n);
    if (lane == 0) {
      e->nruns[row] = ns;
      e->live_cnt[row] = n;
    }
  }
}

// Bound by latency and by the partials' way through memory (64 KB per segment; 16 MB for 256 segments): loads of several
// segments, or of eight tiles' maxima, in flight together (call of 32 rows x 4 segments of 4 tiles 22.0 -> 20.7 us, of
// 128 rows x 2 segments of 64 tiles 163 -> 147 us, against one load at a time); written past the L2 and read without
// leaving a trace there (a step of 32 rows x 16 tiles 18.8 -> 16.5 us, of 72 x 12 24.1 -> 19.5, of 100 x 25 36.1 ->
// 34.6; the stores alone give a third of it, nt in place of sc1 half).  What a workgroup asks for goes out together, not the
// partial O behind the row maxima or the tiles' maxima behind the mask row, and the workgroups with the longer chain, which
// judge, come first: with that, 32 x 16, four steps, 68.9 -> 63.3 us, 72 x 12, three, 58.5 -> 56.6; judging last, the latter
// 59.5, as its loads then wait behind all partial results.  O of two segments at a time in flight: 32 x 16
// 63.5 -> 61.8 us against four (eight 63.7, one 69.8), 72 x 12 56.3 -> 55.6 (60.5, 55.1), 100 x 25 dense, three steps,
// 106.1 -> 101.4, 64 x 64 131.4 -> 130.5: all workgroups ask at the same moment.
// Rows that were cut into segments (FEW, nseg > 1): merges the segments' partial results and judges the tiles.
// Workgroups 0 .. rows-1: one Skip-Mask row each: the tiles' maxima are walked with the running maximum carried over
// (exactly the maximum a single pass would have), the row's mask bits are set and the step's counters added.  Workgroups
// rows .. 5*rows-1: 32 Q rows each, one thread per (row, 8 features): O = sum_s 2^(c (m_s - M)) O_s / sum_s ... .
constexpr int kMergeThreads = 512;
constexpr int kJudged = 64;  // tiles of a row that are judged in one trip to memory; longer rows: two waves per segment
__global__ __launch_bounds__(kMergeThreads) void merge_segments_kernel(const FwdParams p) {
  touch_arguments(sizeof(FwdParams));
  const int tid = threadIdx.x, lane = tid & 63;
  const int nseg = p.nseg;
  if ((int)blockIdx.x >= p.rows_total) {
    const int row = (blockIdx.x - p.rows_total) >> 2, wave = (blockIdx.x - p.rows_total) & 3;
    const int bh = quotient(row, p.Tq, p.per_Tq), i = row - bh * p.Tq;
    const int lq = tid & 31, e = tid >> 5;  // e = 4 * d-block + group of four accumulator registers
    const int qrow = i * kTile + 32 * wave + lq;
    const float* ps = p.seg_stat + (size_t)row * nseg * 2 * kTile + 32 * wave + lq;
    const float* po = p.seg_o + ((size_t)row * nseg * 4 + wave) * 4096 + 256 * e + 4 * lq;
    const float c = p.scale * 1.4426950408889634f;
    constexpr int kAhead = 2;  // segments whose O is in flight together
    float m[kMaxSegments], ls[kMaxSegments], top = kNoMax, l = 0.f;
    f32x4 x[kAhead], y[kAhead];
    auto load_o = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const float* at = po + (size_t)min(s0 + u, nseg - 1) * 4 * 4096;
        x[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(at));
        y[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(at + 128));
      }
    };
    // all segments' row maxima and sums and the first segments' O in flight together
#pragma unroll
    for (int s = 0; s < kMaxSegments; ++s) {
      m[s] = kNoMax;
      if (s / kAhead * kAhead >= nseg) continue;
      m[s] = ps[min(s, nseg - 1) * 2 * kTile];
      ls[s] = ps[min(s, nseg - 1) * 2 * kTile + kTile];
    }
    load_o(0);
#pragma unroll
    for (int s = 0; s < kMaxSegments; ++s) top = fmaxf(top, m[s]);
    float4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s0 = 0; s0 < kMaxSegments; s0 += kAhead) {
      if (s0 >= nseg) break;
      if (s0 > 0) load_o(s0);
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (s0 + u >= nseg || m[s0 + u] == kNoMax) continue;  // a segment without tiles has written no O
        const float f = __builtin_amdgcn_exp2f((m[s0 + u] - top) * c);
        l += f * ls[s0 + u];
        a.x += f * x[u].x; a.y += f * x[u].y; a.z += f * x[u].z; a.w += f * x[u].w;
        b.x += f * y[u].x; b.y += f * y[u].y; b.z += f * y[u].z; b.w += f * y[u].w;
      }
    }
    if (qrow >= p.N) return;
    const float inv = l > 0.f ? 1.f / l : 0.f;
    uint4 o;
    o.x = pack_bf16x2(a.x * inv, a.y * inv);
    o.y = pack_bf16x2(a.z * inv, a.w * inv);
    o.z = pack_bf16x2(b.x * inv, b.y * inv);
    o.w = pack_bf16x2(b.z * inv, b.w * inv);
    const int batch = quotient(bh, p.H, p.per_H);
    uint16_t* out = p.out + (int64_t)batch * p.stride_b + (int64_t)(bh - batch * p.H) * p.stride_h;
    *reinterpret_cast<uint4*>(out + (int64_t)qrow * p.stride_n + 8 * e) = o;
    return;
  }
  constexpr int kPairs = kMergeThreads / 128;
  __shared__ uint64_t fired[2 * kPairs][64];  // per wave (half of a segment's Q rows): tiles that fire for its rows
  const int row = blockIdx.x;
  const int i = row - quotient(row, p.Tq, p.per_Tq) * p.Tq;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = tid & 127, pair = wave >> 1;
  LiveWalk walk;
  int cnt, nruns;
  // the mask row and the segments' row maxima, all in flight together
  const uint64_t skipped = LiveWalk::load(p.bits + (size_t)row * p.W, p.fresh, p.W);
  float seg_max[kMaxSegments];
#pragma unroll
  for (int x = 0; x < kMaxSegments; ++x)
    if (p.Tk > kJudged && (x < 4 || nseg > 4))
      seg_max[x] = p.seg_stat[((size_t)row * nseg + min(x, nseg - 1)) * 2 * kTile + r];
  const bool q_pinned = p.protect_len > 0 && i * kTile < p.protect_start + p.protect_len &&
                        p.protect_start < min(p.N, (i + 1) * kTile);
  uint64_t mine = 0;  // lane w: bits of mask word w
  const bool qvalid = i * kTile + r < p.N;
  const float* mloc = p.seg_mloc + (size_t)row * p.Tk * kTile + r;
  const int start = p.diagonal_first ? i : 0;
  if (p.thr > -INFINITY && !q_pinned && p.Tk <= kJudged) {
    // Short rows: each pair of waves takes a quarter of the row's places in visiting order, whatever the segments were, and
    // asks for the maxima of all of them, skipped or not, before the mask row is here: one trip to memory.  The quarters'
    // maxima meet in LDS.
    constexpr int kEach = kJudged / kPairs;
    __shared__ float quarter[kPairs][kTile];
    const int each = (p.Tk + kPairs - 1) / kPairs, v0 = pair * each, count = min(each, p.Tk - v0);
    const uint64_t dead = (uint32_t)__builtin_amdgcn_readfirstlane((int)skipped) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(skipped >> 32)) << 32;
    auto tile = [&](int u) { return start + v0 + u >= p.Tk ? start + v0 + u - p.Tk : start + v0 + u; };
    float m[kEach], top = -INFINITY;
#pragma unroll
    for (int u = 0; u < kEach; ++u)
      if (u < count) m[u] = mloc[tile(u) * kTile];
#pragma unroll
    for (int u = 0; u < kEach; ++u)
      if (u < count && !(dead >> tile(u) & 1)) top = fmaxf(top, m[u]);
    quarter[pair][r] = top;
    __syncthreads();
    float run = -INFINITY;
    for (int x = 0; x < pair; ++x) run = fmaxf(run, quarter[x][r]);
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      if (u >= count || (dead >> tile(u) & 1)) continue;
      run = fmaxf(run, m[u]);
      if (__all(!qvalid || (m[u] - run) * p.scale <= p.thr) && lane == 0) {
        const bool k_pinned = p.protect_len > 0 && tile(u) * kTile < p.protect_start + p.protect_len &&
                              p.protect_start < min(p.N, (tile(u) + 1) * kTile);
        if (!k_pinned) mine |= 1ull << tile(u);
      }
    }
  } else if (p.thr > -INFINITY && !q_pinned) {
    walk.open(skipped, p.Tk, p.W, start);
    walk.count(cnt, nruns);
    for (int s = pair; s < nseg; s += kPairs) {
      const int t0 = segment_start(cnt, s, nseg), t1 = segment_start(cnt, s + 1, nseg);
      if (t0 == t1) continue;
      float run = -INFINITY;
#pragma unroll
      for (int x = 0; x < kMaxSegments; ++x) run = x < s ? fmaxf(run, seg_max[x]) : run;
      walk.rewind();
      walk.skip(t0);
      constexpr int kAhead = 8;  // tiles whose loads are in flight together
      for (int t = t0; t < t1; t += kAhead) {
        int j[kAhead];
        float m[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          j[u] = u > 0 ? j[u - 1] : 0;
          walk.next(j[u]);
          // (unknown: seen as the tile before where the row has ended, its load became a copy that the others waited for; a
          // step that marks, 100 x 100 110 -> 99 us, 200 x 200 338 -> 316)
          asm volatile("" : "+s"(j[u]));
          m[u] = mloc[(size_t)j[u] * kTile];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          if (t + u >= t1) break;
          run = fmaxf(run, m[u]);
          if (__all(!qvalid || (m[u] - run) * p.scale <= p.thr) && lane == (j[u] >> 6)) {
            const bool k_pinned = p.protect_len > 0 && j[u] * kTile < p.protect_start + p.protect_len &&
                                  p.protect_start < min(p.N, (j[u] + 1) * kTile);
            if (!k_pinned) mine |= 1ull << (j[u] & 63);
          }
        }
      }
    }
  }
  fired[wave][lane] = mine;
  __syncthreads();
  if (wave == 0) {
    uint64_t f = 0;
#pragma unroll
    for (int x = 0; x < kPairs; ++x) f |= fired[2 * x][lane] & fired[2 * x + 1][lane];
    finish_mask_row(*(const_params_ptr)__builtin_amdgcn_kernarg_segment_ptr(), row, lane, skipped, f);
  }
  if (wave == 1 && p.stat_newly && !p.fresh) {
    walk.open(skipped, p.Tk, p.W, start);
    walk.count(cnt, nruns);
    if (lane != 0) return;
    atomicAdd(p.stat_skipped_in, (unsigned long long)(p.Tk - cnt));
    atomicAdd(p.stat_runs, (unsigned long long)nruns);
  }
}

// Few rows: the live tiles of every row of a mask that no call of a handle has left (pick_piece() reads them), one
// thread per row; `arrive`, if not null, is cleared.
__global__ void count_rows_kernel(const uint64_t* bits, int rows, int Tk, int W, uint32_t* live, uint32_t* arrive) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= rows) return;
  int n = 0;
  for (int w = 0; w < W; ++w) n += live_in_word(bits[(size_t)row * W + w], w, Tk);
  live[row] = (uint32_t)n;
  if (arrive) arrive[row] = 0;
}

hipError_t launch_count_rows(const uint64_t* bits, int rows, int Tk, int W, uint32_t* live, uint32_t* arrive,
                             hipStream_t st) {
  hipLaunchKernelGGL(count_rows_kernel, dim3((rows + 63) / 64), dim3(64), 0, st, bits, rows, Tk, W, live, arrive);
  return hipGetLastError();
}

hipError_t launch_clear(uint64_t* bits, size_t words, unsigned long long* stats, size_t nstats, hipStream_t st) {
  size_t n = words > nstats ? words : nstats;
  int blocks = (int)((n + 255) / 256);
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(clear_state_kernel, dim3(blocks), dim3(256), 0, st, bits, words, stats, nstats);
  return hipGetLastError();
}

hipError_t launch_clear_tickets(uint32_t* tickets, int stride, hipStream_t st) {
  hipLaunchKernelGGL(clear_tickets_kernel, dim3(1), dim3(64), 0, st, tickets, stride);
  return hipGetLastError();
}

hipError_t launch_compact(const uint64_t* bits, int rows, int Tq, int Tk, int W, int diagonal_first, int run_stride,
                          uint32_t* runs, uint32_t* nruns, uint32_t* live_cnt, uint32_t* heads_ranked, hipStream_t st) {
  hipLaunchKernelGGL(compact_skiplist, dim3((rows + 4 * kRowsPerWave - 1) / (4 * kRowsPerWave)), dim3(256), 0, st, bits,
                     rows, Tq, Tk, W, diagonal_first, run_stride, runs, nruns, live_cnt, heads_ranked);
  return hipGetLastError();
}

// LDS of prepare_rows_kernel: a 128 x 128 tile, or Tk + 1 bins and one sum per chunk of a head (more than 64 KB for the
// longest sequences), or the dealing's two words per chunk
static size_t prepare_lds_bytes(int Tq, int Tk) {
  const size_t rank = sizeof(uint32_t) * ((size_t)(Tk + 1) + (size_t)((Tq + kChunkRows - 1) / kChunkRows));
  static_assert(128 * kVtRow >= 2 * sizeof(uint32_t) * kDealMax, "dealing");
  return std::max<size_t>(128 * kVtRow, rank);
}

hipError_t launch_prepare_rows(const RowSchedule& sched, const uint16_t* v, uint16_t* vt, int64_t stride_b, int64_t stride_h,
                               int64_t stride_n, int H, int N, hipStream_t st) {
  hipLaunchKernelGGL(prepare_rows_kernel, dim3((unsigned)(sched.BH * (1 + sched.Tk))), dim3(256),
                     prepare_lds_bytes(sched.Tq, sched.Tk), st, sched, v, vt, stride_b, stride_h, stride_n, H, N, sched.Tk);
  return hipGetLastError();
}

constexpr int kQB = 1;  // 32 Q rows per wave, 4 waves per workgroup, 2 workgroups per CU

hipError_t prepare_fwd() {
  const void* fused[] = {reinterpret_cast<const void*>(lite_attn_fwd_kernel<kQB, false, false, false>),
                         reinterpret_cast<const void*>(lite_attn_fwd_kernel<1, true, false, false>),
                         reinterpret_cast<const void*>(lite_attn_fwd_kernel<1, false, true, false>),
                         reinterpret_cast<const void*>(lite_attn_fwd_kernel<1, true, true, false>),
                         reinterpret_cast<const void*>(lite_attn_fwd_kernel<1, false, true, true>),
                         reinterpret_cast<const void*>(lite_attn_fwd_kernel<1, true, true, true>)};
  for (const void* f : fused) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       std::max(kLdsBytes, kPairLdsBytes));
    if (e != hipSuccess) return e;
  }
  return hipFuncSetAttribute(reinterpret_cast<const void*>(prepare_rows_kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)prepare_lds_bytes(16383, 16383));
}

hipError_t launch_schedule_rows(const uint64_t* bits, int rows, int Tk, int W, int per_xcd, uint32_t* slots,
                                uint32_t* xcd_rows, hipStream_t st) {
  hipLaunchKernelGGL(schedule_rows_kernel, dim3(8), dim3(kSchedThreads), 0, st, bits, rows, Tk, W, per_xcd, slots, xcd_rows);
  return hipGetLastError();
}

hipError_t launch_fwd(const FwdParams& p, bool immediate, hipStream_t st) {
  // Workgroups per XCD: one for every segment, piece or row of its share, in order; one for every entry of its list,
  // where these go by place (those past the last row return at once); where rows are drawn, of its share and an eighth
  // more, as an XCD may come to more rows than its list has: not for every entry of a table that has room for unequal
  // lists, since a workgroup that draws in vain costs a counter's round trip too (a later step of 1200 rows x 12 tiles
  // 96 -> 90 us, 8000 x 16 839 -> 822).
  const bool draws = p.tickets && p.resident == kResident, table = p.nseg > 0 && p.scheduled;
  const int rows = (p.rows_total + 7) / 8;
  int places = p.per_xcd;
  if (p.nseg > 0 && !p.tickets)
    places = (std::max(p.rows_total * p.nseg * p.equal_pieces, p.piece_units) + 7) / 8;
  else if (p.nseg > 0 && p.rows_total <= kSchedRows)
    places = !table || draws ? rows + p.cut_rows * (p.cut_pieces - 1) : p.per_xcd - kTableTail;
  const dim3 grid(8 * (draws ? places + places / 8 + 8 : places)), block(Geo<kQB>::kThreads);
  if (p.nseg == 0) {
    if (immediate)
      hipLaunchKernelGGL((lite_attn_fwd_kernel<1, true, false, false>), grid, block, kLdsBytes, st, p);
    else
      hipLaunchKernelGGL((lite_attn_fwd_kernel<kQB, false, false, false>), grid, block, kLdsBytes, st, p);
    return hipGetLastError();
  }
  if (p.pair) {
    if (immediate)
      hipLaunchKernelGGL((lite_attn_fwd_kernel<1, true, true, true>), grid, dim3(512), kPairLdsBytes, st, p);
    else
      hipLaunchKernelGGL((lite_attn_fwd_kernel<1, false, true, true>), grid, dim3(512), kPairLdsBytes, st, p);
  } else if (immediate) {
    hipLaunchKernelGGL((lite_attn_fwd_kernel<1, true, true, false>), grid, block, kLdsBytes, st, p);
  } else {
    hipLaunchKernelGGL((lite_attn_fwd_kernel<1, false, true, false>), grid, block, kLdsBytes, st, p);
  }
  if (p.nseg > 1) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(merge_segments_kernel, dim3(5 * p.rows_total), dim3(kMergeThreads), 0, st, p);
  }
  return hipGetLastError();
}

}  // namespace la
