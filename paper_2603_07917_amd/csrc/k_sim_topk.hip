// Fused similarity search + streaming top-k (the predictor's neighbour search,
// Sec. 3.1: brute-force cosine similarity of prompt embeddings against the
// history store; unit vectors make it an inner product).
//
// GEMM core (shared by the two kernels below). A workgroup of 4 wavefronts
// multiplies one step of 256 history rows by a tile of BQ queries:
// S^T[256 x BQ] = H_step[256 x d] * Q_tile^T with v_mfma_f32_32x32x16_bf16
// (fp32 accumulate). Wave w owns history rows [64w, 64w + 64) of the step and
// all BQ queries. The d axis is walked in 64-wide slices (128-byte row
// pieces) staged through LDS (rows padded to 144 bytes, which keeps the
// 16-byte MFMA operand reads free of bank conflicts); the next slice is
// fetched into registers while the current one is multiplied. The scores of
// a step depend only on (step, query tile), so both kernels compute
// bit-identical scores for the same (query, row) pair.
//
// threshold_sample_kernel: for every query, the maxima of disjoint 16-row
//   groups over a sample of steps (every SR-th step). The k-th largest
//   group maximum is a score reached by k distinct history rows, hence a
//   valid lower bound theta0 on the query's k-th best score.
// sim_topk_kernel: one workgroup owns a query tile and a chunk of history
//   rows. After each step, a lane compares its scores with the query's
//   thresholds (>= theta0, and > the k-th key of the chunk list so far: rows
//   come in index order, so a later equal score loses the tie), appends the
//   survivors as 64-bit keys (monotone score bits, then ~index) to a per-query
//   LDS buffer at deterministic positions (in rounds of 64 with merges in
//   between when a step brings more), and the wave owning the query folds
//   full buffers into the query's descending list with a bitonic merge. The
//   lists end in the partial buffer [Q][chunks][KL].
#include <algorithm>
#include <atomic>

#include "sage.h"
#include "sage_device.hpp"
#include "sage_internal.hpp"

namespace sage {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int kThreads = 256;
constexpr int kStepRows = 256;     // history rows per step (64 per wave)
constexpr int kKT = 64;            // d elements per LDS slice
constexpr int kRowE = kKT + 8;     // padded LDS row: 72 bf16 = 144 bytes
// Per-query candidate buffer: 64 keys, or 32 for 128-query tiles (LDS budget).
template <int NQT> struct CapOf { static constexpr int value = NQT >= 4 ? 32 : 64; };

template <int NQT>
struct Core {
  static constexpr int BQ = 32 * NQT;
  static constexpr int A_LD = kStepRows * kKT / 8 / kThreads;    // 16-byte loads / thread
  static constexpr int B_CHUNKS = BQ * kKT / 8;
  static constexpr int B_LD = (B_CHUNKS + kThreads - 1) / kThreads;
  uint4 ra[A_LD];
  uint4 rb[B_LD];

  // Loads are unconditional (rows clamped into range) so that no branch sits
  // around them; only the zero-fill of columns past d is a select. Rows past
  // h_end and queries past Q carry real but unused data (masked later).
  // The query whose columns this thread's c-th load of a slice fetches: slot
  // (that load's row) of the tile.
  static __device__ __forceinline__ int slot(int c) { return min(c * kThreads + (int)threadIdx.x, B_CHUNKS - 1) >> 3; }
  __device__ __forceinline__ void load(const EmbView& hist, int h0, int h_last, const EmbView& queries,
                                       const int (&q_of)[B_LD], int d, int kt) {
    const int tid = threadIdx.x;
    const int k0 = kt * kKT;
#pragma unroll
    for (int c = 0; c < A_LD; ++c) {
      const int f = c * kThreads + tid;
      const int row = f >> 3, col = k0 + (f & 7) * 8;
      const int h = min(h0 + row, h_last);
      const uint4 v = *reinterpret_cast<const uint4*>(emb_at(hist, h, min(col, d - 8)));
      ra[c] = col < d ? v : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < B_LD; ++c) {
      const int f = min(c * kThreads + tid, B_CHUNKS - 1);
      const int col = k0 + (f & 7) * 8;
      const uint4 v = *reinterpret_cast<const uint4*>(emb_at(queries, q_of[c], min(col, d - 8)));
      rb[c] = col < d ? v : make_uint4(0, 0, 0, 0);
    }
  }
  __device__ __forceinline__ void store(uint16_t* a_tile, uint16_t* b_tile) const {
    const int tid = threadIdx.x;
#pragma unroll
    for (int c = 0; c < A_LD; ++c) {
      const int f = c * kThreads + tid;
      *reinterpret_cast<uint4*>(a_tile + (f >> 3) * kRowE + (f & 7) * 8) = ra[c];
    }
#pragma unroll
    for (int c = 0; c < B_LD; ++c) {
      const int f = c * kThreads + tid;
      if (B_CHUNKS % kThreads == 0 || f < B_CHUNKS)
        *reinterpret_cast<uint4*>(b_tile + (f >> 3) * kRowE + (f & 7) * 8) = rb[c];
    }
  }
};

template <int NQT>
__device__ __forceinline__ void mfma_slice(floatx16 (&acc)[2][NQT], const uint16_t* a_tile,
                                           const uint16_t* b_tile, int w, int l32, int half) {
  const uint16_t* as = a_tile + (64 * w + l32) * kRowE + half * 8;
  const uint16_t* bs = b_tile + l32 * kRowE + half * 8;
#pragma unroll
  for (int kk = 0; kk < kKT / 16; ++kk) {
    bf16x8 af[2], bfr[NQT];
#pragma unroll
    for (int u = 0; u < 2; ++u) af[u] = *reinterpret_cast<const bf16x8*>(as + 32 * u * kRowE + kk * 16);
#pragma unroll
    for (int t = 0; t < NQT; ++t) bfr[t] = *reinterpret_cast<const bf16x8*>(bs + 32 * t * kRowE + kk * 16);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int t = 0; t < NQT; ++t)
        acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[u], bfr[t], acc[u][t], 0, 0, 0);
  }
}

// Scores of one step: acc[u][t][v] = S[h][q] with
//   h = h0 + 64w + 32u + 8(v/4) + 4*half + (v%4),  q = the tile's query 32t + l32
// (q_of: those whose columns this thread loads).
template <int NQT>
__device__ __forceinline__ void gemm_step(floatx16 (&acc)[2][NQT], const EmbView& hist, int h0, int h_end,
                                          const EmbView& queries, const int (&q_of)[Core<NQT>::B_LD], int d,
                                          uint16_t* a_tile, uint16_t* b_tile) {
  const int lane = (int)lane_id();
  const int w = threadIdx.x / kWave;
  const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int t = 0; t < NQT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[u][t][v] = 0.0f;
  const int nk = (d + kKT - 1) / kKT;
  const int h_last = h_end - 1;
  Core<NQT> core;
  core.load(hist, h0, h_last, queries, q_of, d, 0);
  for (int kt = 0; kt + 1 < nk; ++kt) {
    __syncthreads();
    core.store(a_tile, b_tile);
    __syncthreads();
    core.load(hist, h0, h_last, queries, q_of, d, kt + 1);
    mfma_slice<NQT>(acc, a_tile, b_tile, w, l32, half);
  }
  __syncthreads();
  core.store(a_tile, b_tile);
  __syncthreads();
  mfma_slice<NQT>(acc, a_tile, b_tile, w, l32, half);
}

__device__ __forceinline__ uint64_t umax64(uint64_t a, uint64_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint64_t umin64(uint64_t a, uint64_t b) { return a > b ? b : a; }

// Fold `n_buf` (<= 64) unsorted keys of `buf` into the descending list of KL
// keys and return the list key at position k-1 (the same value in every lane).
template <int KL>
__device__ uint64_t merge_into_list(uint64_t* list, const uint64_t* buf, int n_buf, int k) {
  constexpr int S = KL / 64;
  const int lane = (int)lane_id();
  uint64_t lv[S];
#pragma unroll
  for (int s = 0; s < S; ++s) lv[s] = list[s * 64 + lane];
  uint64_t b = lane < n_buf ? buf[lane] : kPadKey;
  const uint64_t br = wave_sort64(b, false);          // ascending along the lanes
  lv[S - 1] = umax64(lv[S - 1], br);                  // bitonic over the KL positions
#pragma unroll
  for (int st = S / 2; st >= 1; st >>= 1) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if ((s & st) == 0) {
        const uint64_t x = lv[s], y = lv[s + st];
        lv[s] = umax64(x, y);
        lv[s + st] = umin64(x, y);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
#pragma unroll
    for (int stride = 32; stride > 0; stride >>= 1) lv[s] = cx_lanes(lv[s], stride, true);
    list[s * 64 + lane] = lv[s];
  }
  const int ks = (k - 1) >> 6, kl = (k - 1) & 63;
  uint64_t sel = lv[0];
#pragma unroll
  for (int s = 1; s < S; ++s) if (s == ks) sel = lv[s];
  return lane_value_u64(sel, kl);
}

// ------------------------------------------------------------------------
// Sampled group maxima: one workgroup per (query tile, sampled step).
// gm[q][s][g] for the 16 groups of 16 rows of a step; -inf past N.
// ------------------------------------------------------------------------
template <int NQT>
__global__ void __launch_bounds__(kThreads, 1) threshold_sample_kernel(
    EmbView queries, int Q, EmbView hist, int N, int d,
    int sample_every, int n_samples, float* __restrict__ gm) {
  constexpr int BQ = 32 * NQT;
  __shared__ __align__(16) uint16_t a_tile[kStepRows * kRowE];
  __shared__ __align__(16) uint16_t b_tile[BQ * kRowE];
  const int q0 = blockIdx.x * BQ;
  const int s = blockIdx.y;
  const int h0 = s * sample_every * kStepRows;
  const int h_end = min(N, h0 + kStepRows);
  int q_of[Core<NQT>::B_LD];
#pragma unroll
  for (int c = 0; c < Core<NQT>::B_LD; ++c) q_of[c] = min(q0 + Core<NQT>::slot(c), Q - 1);
  floatx16 acc[2][NQT];
  gemm_step<NQT>(acc, hist, h0, h_end, queries, q_of, d, a_tile, b_tile);

  const int lane = (int)lane_id();
  const int w = threadIdx.x / kWave;
  const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
  for (int t = 0; t < NQT; ++t) {
    const int q = q0 + 32 * t + l32;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float m = -__builtin_inff();
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int h = h0 + 64 * w + 32 * u + 8 * (v >> 2) + 4 * half + (v & 3);
        if (h < h_end) m = fmaxf(m, acc[u][t][v]);
      }
      if (q < Q) gm[((size_t)q * n_samples + s) * 16 + w * 4 + half * 2 + u] = m;
    }
  }
}

// ------------------------------------------------------------------------
// Main kernel.
// ------------------------------------------------------------------------
template <int NQT, int KL>
struct TopkSmem {
  static constexpr int BQ = 32 * NQT;
  static constexpr int kCap = CapOf<NQT>::value;
  uint64_t list[BQ * KL];
  uint64_t buf[BQ * kCap];
  uint16_t a_tile[kStepRows * kRowE];
  uint16_t b_tile[BQ * kRowE];
  float theta[BQ];
  float theta0[BQ];
  int fill[BQ];
  int tot[BQ];
  int cnt[BQ * 8];
  int rounds;
  int query[BQ];                           // the tile's queries
  int wave_n[kThreads / kWave];
};

// The flagged queries of ranks q0 .. q0 + BQ - 1 among all flagged ones, in
// order, to sm.query. Every thread of the workgroup calls it.
template <int NQT, int KL>
__device__ __forceinline__ void gather_flagged(TopkSmem<NQT, KL>& sm, const int* __restrict__ flags, int Q, int q0) {
  constexpr int BQ = 32 * NQT;
  const int tid = threadIdx.x;
  const int w = tid / kWave;
  const uint64_t below = (1ull << lane_id()) - 1ull;
  int found = 0;
  for (int base = 0; base < Q && found < q0 + BQ; base += kThreads) {
    const bool on = base + tid < Q && flags[base + tid] != kNotFlagged;
    const uint64_t mask = __ballot(on);
    if (lane_id() == 0) sm.wave_n[w] = __popcll(mask);
    __syncthreads();
    int rank = found + __popcll(mask & below);
#pragma unroll
    for (int i = 0; i < kThreads / kWave; ++i) {
      if (i < w) rank += sm.wave_n[i];
      found += sm.wave_n[i];
    }
    if (on && rank >= q0 && rank < q0 + BQ) sm.query[rank - q0] = base + tid;
    __syncthreads();                       // wave_n read; query complete
  }
}

// One (query tile, history chunk) of the list search: of all Q queries, or as
// the exact fallback of the n_flagged queries that are flagged, whose tiles
// then hold no others.
template <int NQT, int KL, bool kFallback>
__device__ __forceinline__ void list_tile(TopkSmem<NQT, KL>& sm, EmbView queries, int Q, EmbView hist, int N,
                                          int d, int k, int chunk_rows, int n_chunks, int q_tiles,
                                          const float* __restrict__ theta0, const int* __restrict__ only_flagged,
                                          int n_flagged, uint64_t* __restrict__ partial, const int b) {
  constexpr int BQ = 32 * NQT;
  constexpr int QPW = BQ / 4;              // queries merged by each wave
  constexpr int kCap = CapOf<NQT>::value;

  // Block -> (query tile, chunk). When the chunks split evenly over the 8
  // XCDs, the query tiles of one chunk are dispatched to the same XCD so that
  // its history rows are shared through that XCD's L2.
  int qt, chunk;
  if (n_chunks % 8 == 0) {
    const int x = b & 7, slot = b >> 3;
    chunk = x + 8 * (slot / q_tiles);
    qt = slot % q_tiles;
  } else {
    chunk = b / q_tiles;
    qt = b % q_tiles;
  }
  const int tid = threadIdx.x;
  const int lane = (int)lane_id();
  const int w = tid / kWave;
  const int l32 = lane & 31, half = lane >> 5;
  const int q0 = qt * BQ;
  const int h_begin = chunk * chunk_rows;
  const int h_end = min(N, h_begin + chunk_rows);

  const int n_q = kFallback ? n_flagged : Q;           // queries in all tiles
  if (kFallback) {
    for (int i = tid; i < BQ; i += kThreads) sm.query[i] = 0;
    __syncthreads();
    gather_flagged(sm, only_flagged, Q, q0);
  }
  auto query = [&](int i) { return kFallback ? sm.query[i] : min(q0 + i, Q - 1); };   // of slot i
  int q_of[Core<NQT>::B_LD];
#pragma unroll
  for (int c = 0; c < Core<NQT>::B_LD; ++c) q_of[c] = query(Core<NQT>::slot(c));

  for (int i = tid; i < BQ * KL; i += kThreads) sm.list[i] = kPadKey;
  for (int i = tid; i < BQ; i += kThreads) {
    sm.theta[i] = -__builtin_inff();
    // As the fallback: the threshold again for a query that has more candidates
    // than its arrays hold (50,000 equal rows of 100,000, 300 queries of which
    // 100 are equal to them, k = 128, d = 384: 852 us without it). It is a bound
    // that k of this query's scores reach; only where too few did, it is not.
    const int q = query(i);
    const bool bound = theta0 && q0 + i < n_q && (!kFallback || only_flagged[q] == kOverflowed);
    sm.theta0[i] = bound ? theta0[q] : -__builtin_inff();
    sm.fill[i] = 0;
  }

  for (int h0 = h_begin; h0 < h_end; h0 += kStepRows) {
    floatx16 acc[2][NQT];
    const int step_end = min(h_end, h0 + kStepRows);
    gemm_step<NQT>(acc, hist, h0, step_end, queries, q_of, d, sm.a_tile, sm.b_tile);

    // ---------------- filter, rank, append, merge ----------------
    // One compare per score: s >= theta0 and s > theta  <=>  s > max(below(theta0), theta),
    // where below(x) is the largest float under x. Rows past the chunk end
    // (only in a chunk's last step) are masked out of the candidate bits.
    const bool full_step = step_end == h0 + kStepRows;
    float thr[NQT];
    uint32_t bits[NQT];
    int my_cnt[NQT];
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
      const int ql = 32 * t + l32;
      thr[t] = fmaxf(float_below(sm.theta0[ql]), sm.theta[ql]);
      // Bit i = [s_i > thr] is the sign bit of thr - s_i, shifted in with
      // one funnel shift per score.
      uint32_t m = 0;
#pragma unroll
      for (int u = 1; u >= 0; --u)
#pragma unroll
        for (int v = 15; v >= 0; --v)
          m = __builtin_amdgcn_alignbit(m, __float_as_uint(thr[t] - acc[u][t][v]), 31);
      if (!full_step) {
        // Bit i = 16 u + v is row h0 + 64 w + 4 half + 8 (i / 4) + i % 4:
        // rows grow with i, so the rows inside the step are the lowest bits.
        const int c = min(max(step_end - h0 - 64 * w - 4 * half, 0), 64);
        const int n_in = 4 * (c >> 3) + min(c & 7, 4);
        m &= n_in >= 32 ? ~0u : (1u << n_in) - 1u;
      }
      if (q0 + ql >= n_q) m = 0;
      bits[t] = m;
      my_cnt[t] = __popc(m);
      sm.cnt[ql * 8 + 2 * w + half] = my_cnt[t];
    }
    if (tid == 0) sm.rounds = 1;
    __syncthreads();
    if (tid < BQ) {
      int s = sm.fill[tid];
#pragma unroll
      for (int j = 0; j < 8; ++j) s += sm.cnt[tid * 8 + j];
      sm.tot[tid] = s;
      const int r = (s + kCap - 1) / kCap;
      if (r > 1) atomicMax(&sm.rounds, r);
    }
    __syncthreads();
    const int rounds = sm.rounds;
    int base[NQT];
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
      const int ql = 32 * t + l32;
      int bb = sm.fill[ql];
      for (int j = 0; j < 2 * w + half; ++j) bb += sm.cnt[ql * 8 + j];
      base[t] = bb;
    }
    for (int r = 0; r < rounds; ++r) {
      const int lo = r * kCap, hi = lo + kCap;
#pragma unroll
      for (int t = 0; t < NQT; ++t) {
        const int ql = 32 * t + l32;
        if (my_cnt[t] == 0 || base[t] + my_cnt[t] <= lo || base[t] >= hi) continue;
        int g = base[t];
        uint32_t m = bits[t];
        while (m) {
          const int i = __ffs(m) - 1;
          m &= m - 1;
          if (g >= lo && g < hi) {
            const int u = i >> 4, v = i & 15;
            const int h = h0 + 64 * w + 32 * u + 8 * (v >> 2) + 4 * half + (v & 3);
            float sv = 0.0f;
#pragma unroll
            for (int uu = 0; uu < 2; ++uu)
#pragma unroll
              for (int vv = 0; vv < 16; ++vv)
                if (16 * uu + vv == i) sv = acc[uu][t][vv];
            sm.buf[ql * kCap + (g - lo)] = make_key(sv, (uint32_t)h);
          }
          ++g;
        }
      }
      __syncthreads();
      if (r + 1 < rounds) {
        for (int j = 0; j < QPW; ++j) {
          const int ql = w * QPW + j;
          if (sm.tot[ql] > hi) {
            const uint64_t kth = merge_into_list<KL>(&sm.list[ql * KL], &sm.buf[ql * kCap], kCap, k);
            if (lane == 0) sm.theta[ql] = key_sim(kth);
          }
        }
        __syncthreads();
      }
    }
    if (tid < BQ) {
      const int s = sm.tot[tid];
      sm.fill[tid] = s > 0 ? s - kCap * ((s - 1) / kCap) : 0;
    }
    // theta / fill are next read after the following step's barriers.
  }

  __syncthreads();
  for (int j = 0; j < QPW; ++j) {
    const int ql = w * QPW + j;
    const int f = sm.fill[ql];
    if (f > 0) merge_into_list<KL>(&sm.list[ql * KL], &sm.buf[ql * kCap], f, k);
  }
  __syncthreads();
  for (int i = tid; i < BQ * KL; i += kThreads) {
    const int ql = i / KL, e = i - ql * KL;
    if (q0 + ql < n_q) partial[((size_t)query(ql) * n_chunks + chunk) * KL + e] = sm.list[i];
  }
}

template <int NQT, int KL, bool kFallback>
__global__ void __launch_bounds__(kThreads, 1) sim_topk_kernel(
    EmbView queries, int Q, EmbView hist, int N, int d,
    int k, int chunk_rows, int n_chunks, int q_tiles, const float* __restrict__ theta0,
    const int* __restrict__ only_flagged, const uint32_t* __restrict__ flag_word,
    uint64_t* __restrict__ partial) {
  __shared__ __align__(16) TopkSmem<NQT, KL> sm;
  // As the exact fallback: nothing to do unless a query of this call was
  // flagged (the flagging kernel counts them in the word), and the tiles of
  // those that were.
  const int n_flagged = kFallback ? (int)*flag_word : 0;
  if (kFallback) q_tiles = (n_flagged + 32 * NQT - 1) / (32 * NQT);
  // Tiles b = blockIdx.x, + gridDim.x, ... (one each for the full search).
  for (int b = blockIdx.x; b < q_tiles * n_chunks; b += gridDim.x) {
    __syncthreads();                         // the previous tile's LDS reads are done
    list_tile<NQT, KL, kFallback>(sm, queries, Q, hist, N, d, k, chunk_rows, n_chunks, q_tiles, theta0, only_flagged,
                       n_flagged, partial, b);
  }
}



// theta0: the k-th largest of a query's m (<= 512 * 16) group maxima, held
// in registers as monotone key bits (VPL per lane; past m: key 0, below every
// real score). theta0 is the largest key T with at least k keys >= T, built
// bit by bit from the top: each bit costs one compare per key and a sum. That
// T is exactly the k-th largest key. Every key lies in [lo, hi], and so does
// the answer: the bits above the highest one where lo and hi differ are fixed
// from the start.
//
// WAVES = 1: one wavefront per query, four queries per workgroup (many
// queries). WAVES > 1: one workgroup of WAVES wavefronts per query, the sums
// completed through LDS (few queries, where one wave per query would leave
// the chip idle and each wave latency-bound).
template <int VPL, int WAVES>
__global__ void __launch_bounds__(256 * (WAVES > 1 ? WAVES / 4 : 1)) threshold_select_kernel(
    const float* __restrict__ gm, int Q, int m, int k, float* __restrict__ theta0, int* __restrict__ clear) {
  __shared__ uint32_t part[2][WAVES > 1 ? WAVES : 1];
  __shared__ uint32_t ext[2][WAVES > 1 ? WAVES : 1];
  const int lane = (int)lane_id();
  const int w = (int)(threadIdx.x / kWave);
  const int q = WAVES > 1 ? (int)blockIdx.x : (int)(blockIdx.x * (blockDim.x / kWave) + w);
  if (q >= Q) return;                                   // whole wavefronts (WAVES = 1 only)
  const float* src = gm + (size_t)q * m;
  const int first = WAVES > 1 ? w * VPL * kWave : 0;    // this wave's keys: first + i * 64 + lane
  uint32_t key[VPL];
  uint32_t kmax = 0, kmin = 0xffffffffu;
#pragma unroll
  for (int i = 0; i < VPL; ++i) {
    const int e = first + i * kWave + lane;
    key[i] = e < m ? f32_order_bits(src[e]) : 0u;
    kmax = max(kmax, key[i]);
    if (e < m) kmin = min(kmin, key[i]);
  }
  uint32_t hi = wave_max_dpp_u32(kmax), lo = wave_min_dpp_u32(kmin);
  if (WAVES > 1) {
    if (lane == 0) { ext[0][w] = hi; ext[1][w] = lo; }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WAVES; ++i) { hi = max(hi, ext[0][i]); lo = min(lo, ext[1][i]); }
  }
  const int top = hi == lo ? -1 : 31 - __clz(hi ^ lo);
  uint32_t T = top < 0 ? hi : hi & ~((2u << top) - 1u);
  for (int bit = top; bit >= 0; --bit) {
    const uint32_t c = T | (1u << bit);
    uint32_t n0 = 0, n1 = 0;
#pragma unroll
    for (int i = 0; i < VPL; i += 2) {
      n0 += key[i] >= c ? 1u : 0u;
      if (i + 1 < VPL) n1 += key[i + 1] >= c ? 1u : 0u;
    }
    uint32_t n = wave_sum_dpp_u32(n0 + n1);
    if (WAVES > 1) {                                    // partials alternate buffers: one barrier per bit
      if (lane == 0) part[bit & 1][w] = n;
      __syncthreads();
      n = 0;
#pragma unroll
      for (int i = 0; i < WAVES; ++i) n += part[bit & 1][i];
    }
    if (n >= (uint32_t)k) T = c;
  }
  if (lane == 0 && (WAVES == 1 || w == 0)) {
    theta0[q] = k <= m ? f32_from_order_bits(T) : -__builtin_inff();
    if (clear) clear[q] = 0;                            // the next kernel's per-query counter
  }
}
// ========================================================================
// Filtered path.
//
// Ring core: a workgroup multiplies 256 history rows by kBQ = 64 WQ queries
// per step with 2 WQ waves; wave w = wh * WQ + wq owns the 128 x 64 block of
// rows wh and queries wq (4 x 2 MFMA 32x32x16 tiles, 128 accumulators). The d
// axis is walked in 32-wide slices held in a ring of LDS stages (256 + kBQ
// rows x 64 bytes each). Stages are filled by direct global->LDS loads (16
// bytes per lane, no registers), kStages - 1 slices ahead of the MFMAs and
// straight across step boundaries, so the pipeline never drains between
// steps. One barrier per slice.
//
// Two waves per SIMD: the epilogue (one subtraction and one funnel shift per
// score, and the picking of survivors) is bound by VALU issue, and one wave
// alone issues only every 7 to 7.5 cycles where the SIMD takes one every 4;
// with 256 registers a wave the accumulators are also plain VGPRs, so that the
// epilogue reads them in place instead of copying each from an AGPR. Against
// four waves of 128 x 128 blocks in AGPRs (same tile, 1.5x fewer LDS operand
// reads), same box: 30.43 -> 29.55 ms at 16,384 x 1M x 1024 (fed by the
// last-level cache), 1.590 -> 1.449 ms at 4,096 x 262,144 x 768, 174 -> 149 us
// at 1,001 x 100,003 x 384 (whole decisions).
// ========================================================================
namespace ring {

constexpr int kKT = 32;                          // bf16 columns per slice
constexpr int kRows = 256;                       // history rows per step
template <int WQ>
struct Shape {
  static constexpr int kWaves = 2 * WQ;
  static constexpr int kThreads = kWave * kWaves;
  static constexpr int kBQ = 64 * WQ;            // queries per tile
  // 256 queries: four stages (128 KiB), one workgroup of eight waves per CU.
  // 128 queries: three stages (72 KiB), two workgroups of four waves per CU.
  static constexpr int kStages = WQ == 4 ? 4 : 3;
  static constexpr int kStageBytes = (kRows + kBQ) * kKT * 2;
  static constexpr int kHL = kRows / 16 / kWaves;   // history loads per wave and slice
  static constexpr int kQL = kBQ / 16 / kWaves;     // query loads per wave and slice
  static constexpr int kLoads = kHL + kQL;
  static constexpr int kAhead = kStages - 1;     // slices in flight
};

// 16-byte chunk c (0..3) of LDS row r (64 bytes) is stored at position
// c ^ swz(r). An MFMA operand read has 16 lanes reading one chunk of 16
// consecutive rows per cycle; four rows fill the 64 four-byte banks, and
// swz = (r / 4) % 4 gives the four rows that share banks four different
// positions (measured: no bank conflicts, against one in three LDS cycles
// for the unswizzled layout).
__device__ __forceinline__ int swz(int r) { return (r >> 2) & 3; }

// LDS[m0 + 16*lane] = 16 bytes at base + off (gfx950 global_load_lds_dwordx4).
// Issued from inline assembly so that the compiler does not serialise LDS
// reads of other stages behind it; completion is tracked with wait_loads.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t off, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(base), "s"(m0) : "memory", "m0");
}
// The same when the wave-uniform `enabled` is non-zero, else nothing. The
// test is a branch inside the assembly, which keeps the surrounding MFMA
// sequence in one basic block.
__device__ __forceinline__ void load_to_lds_if(const void* base, uint32_t off, uint32_t m0, int enabled) {
  asm volatile("s_cmp_eq_u32 %3, 0\n\ts_cbranch_scc1 1f\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %0, %1\n1:"
               :: "v"(off), "s"(base), "s"(m0), "s"(enabled) : "memory", "m0", "scc");
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
// Waits until at most n (0 to 2) slices of this wave's loads are in flight,
// and with `half` half a slice more (then n is 0 or 1).
template <int kLoads>
__device__ __forceinline__ void wait_slices(int n, bool half) {
  if (half) {
    if (n <= 0) wait_loads<kLoads / 2>();
    else wait_loads<kLoads + kLoads / 2>();
  } else {
    if (n <= 0) wait_loads<0>();
    else if (n == 1) wait_loads<kLoads>();
    else wait_loads<2 * kLoads>();
  }
}
// Workgroup barrier that first retires this wave's LDS reads. The wait is the
// compiler's own instruction (lgkmcnt(0), other counters untouched), so its
// bookkeeping of outstanding LDS reads stays exact after the barrier.
__device__ __forceinline__ void barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);
  asm volatile("s_barrier" ::: "memory");
}

struct Frags {
  bf16x8 a[4], b[2];
};

// Runs steps h0 = h_first + j * h_stride (j < n_steps) of query tile q0 and
// calls epi(acc, h0, step_end) after each, step_end = min(h_limit, h0 + 256),
// with acc[u][t][v] = S[h][q] for
//   h = h0 + 128 wh + 32 u + 8 (v / 4) + 4 half + v % 4,  q = q0 + 64 wq + 32 t + l32.
// Rows past N - 1 and queries past Q - 1 are read clamped (their scores are
// meaningless and must be masked by the caller). Requires d % 32 == 0.
template <int WQ, class Epi>
__device__ __forceinline__ void sweep(const EmbView& hist, int N, int h_first, int h_stride, int n_steps,
                                      int h_limit, const EmbView& queries, int Q, int q0, int d, char* lds,
                                      Epi& epi) {
  using S = Shape<WQ>;
  constexpr int kLoads = S::kLoads, kHL = S::kHL, kQL = S::kQL, kAhead = S::kAhead;
  constexpr int kGap = 16 / kLoads;             // MFMAs between two loads of a half slice
  constexpr int kStages = S::kStages, kStageBytes = S::kStageBytes;
  static_assert(kLoads % 2 == 0 && (kAhead == 2 || kAhead == 3), "the waits below: half slices, at most two whole ones");
  const int lane = (int)lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wh = w / WQ, wq = w % WQ;
  const int l32 = lane & 31, half = lane >> 5;
  const int nk = d / kKT;
  const int total = n_steps * nk;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

  // Loader: every wave moves kHL pieces of 16 history rows and kQL pieces of
  // 16 query rows per slice; lane l carries chunk (l & 3) ^ swz of row l / 4
  // of a piece (swz of those rows is (l / 16) % 4 for every piece).
  const int rh = 16 * kHL * w + (lane >> 2), rq = 16 * kQL * w + (lane >> 2);
  const uint32_t cb = (uint32_t)(((lane & 3) ^ swz(lane >> 2)) * 16);
  const uint32_t h_row_bytes = (uint32_t)(hist.row * 2), q_row_bytes = (uint32_t)(queries.row * 2);
  const long long h_slice_bytes = hist.panel * 2, q_slice_bytes = queries.panel * 2;
  int ld_step = 0, ld_kt = 0;
  const char* hsrc = nullptr;                 // sources of slice ld_kt of step ld_step
  const char* const qsrc0 = reinterpret_cast<const char*>(emb_at(queries, q0, 0));
  const char* qsrc = qsrc0;
  uint32_t hoff[kHL], qoff[kQL];              // per-lane byte offsets within a slice
#pragma unroll
  for (int i = 0; i < kQL; ++i) qoff[i] = (uint32_t)min(rq + 16 * i, Q - 1 - q0) * q_row_bytes + cb;
  auto next_source = [&]() {                  // at the first slice of step ld_step
    const int base_row = h_first + ld_step * h_stride;
    hsrc = reinterpret_cast<const char*>(emb_at(hist, base_row, 0));
    qsrc = qsrc0;
    const int last = N - 1 - base_row;
#pragma unroll
    for (int i = 0; i < kHL; ++i) hoff[i] = (uint32_t)min(rh + 16 * i, last) * h_row_bytes + cb;
  };
  // Load i of the next slice into a stage: history pieces first, then queries.
  const uint32_t h_lds = lds0 + (uint32_t)(w * kHL * 1024);
  const uint32_t q_lds = lds0 + (uint32_t)((kRows / 16 + w * kQL) * 1024);
  auto issue_one = [&](int stage, int i, bool always, int enabled) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(stage * kStageBytes) + (i < kHL ? h_lds + (uint32_t)i * 1024u : q_lds + (uint32_t)(i - kHL) * 1024u));
    const char* src = i < kHL ? hsrc : qsrc;
    const uint32_t off = i < kHL ? hoff[i < kHL ? i : 0] : qoff[i < kHL ? 0 : i - kHL];
    if (always) load_to_lds(src, off, m0);
    else load_to_lds_if(src, off, m0, __builtin_amdgcn_readfirstlane(enabled));
  };
  auto advance = [&]() {
    hsrc += h_slice_bytes;
    qsrc += q_slice_bytes;
    if (++ld_kt == nk) {
      ld_kt = 0;
      ++ld_step;
      if (ld_step < n_steps) next_source();
    }
  };
  next_source();

  // Operand reads: A = history rows 128 wh + 32 u + l32, B = query rows
  // 256 + 64 wq + 32 t + l32; k chunk 2 kk + half of the slice.
  uint32_t a_off[2], b_off[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const uint32_t pos = (uint32_t)(((2 * kk + half) ^ swz(l32)) * 16);
    a_off[kk] = (uint32_t)((128 * wh + l32) * 64) + pos;
    b_off[kk] = (uint32_t)((kRows + 64 * wq + l32) * 64) + pos;
  }
  // Piece p of the fragments in the order of use: B0, A0, B1, A1, A2, A3.
  auto read_piece = [&](int st, int kk, int p, Frags& f) {
    const char* stage = lds + st * kStageBytes;
    if (p == 0) f.b[0] = *reinterpret_cast<const bf16x8*>(stage + b_off[kk]);
    else if (p == 2) f.b[1] = *reinterpret_cast<const bf16x8*>(stage + b_off[kk] + 2048);
    else {
      const int u = p == 1 ? 0 : p - 2;
      f.a[u] = *reinterpret_cast<const bf16x8*>(stage + a_off[kk] + u * 2048);
    }
  };

  __syncthreads();                              // earlier users of the LDS are done
  const int pre = min(kAhead, total);
  for (int g = 0; g < pre; ++g) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) issue_one(g, i, true, 1);
    advance();
  }
  wait_slices<kLoads>(pre - 1, false);          // slice 0 has landed
  barrier();
  Frags f0, f1;
#pragma unroll
  for (int p = 0; p < 6; ++p) read_piece(0, 0, p, f0);
  int g = 0, st = 0;                            // slice and its stage (g % kStages)
  for (int step = 0; step < n_steps; ++step) {
    floatx16 acc[4][2];
    // One slice: f0 holds its first 16 columns on entry; on exit f0 holds the
    // first 16 columns of slice g + 1 (past the last slice those reads fetch
    // a stale stage, which is never used).
    //  * The fragment reads are spread over the MFMAs, one after each of the
    //    first six of a half, pinned there with scheduling groups: issued as
    //    one burst next to their consumers, the compiler waits on them and
    //    the matrix pipe drains.
    //  * The loads of slice g + kAhead (whose stage was last read in slice
    //    g - 1) go out half of them in each half, which keeps the address unit
    //    evenly busy.
    auto slice = [&](bool first, bool steady) {
      const int more = steady ? 1 : (g + kAhead < total);
      const int st_load = st == 0 ? kStages - 1 : st - 1;         // stage of slice g + kAhead
      const int st_next = st == kStages - 1 ? 0 : st + 1;         // stage of slice g + 1
      const floatx16 zero = {};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int u = j >> 1, t = j & 1;
        acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f0.a[u], f0.b[t], first ? zero : acc[u][t], 0, 0, 0);
        if (j < 6) read_piece(st, 1, j, f1);
        if ((j + 1) % kGap == 0 && (j + 1) / kGap <= kLoads / 2) issue_one(st_load, (j + 1) / kGap - 1, steady, more);
      }
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      // The half's last MFMAs stay before the barrier, so the matrix pipe has
      // work queued while the wave waits for its reads and for the other waves.
      __builtin_amdgcn_sched_barrier(0);
      if (steady) wait_loads<(kAhead - 2) * kLoads + kLoads / 2>();
      else wait_slices<kLoads>(min(kAhead - 2, max(0, total - 2 - g)), more != 0);
      barrier();
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int u = j >> 1, t = j & 1;
        acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1.a[u], f1.b[t], acc[u][t], 0, 0, 0);
        if (j < 6) read_piece(st_next, 0, j, f0);
        if ((j + 1) % kGap == 0 && (j + 1) / kGap <= kLoads / 2)
          issue_one(st_load, kLoads / 2 + (j + 1) / kGap - 1, steady, more);
      }
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      if (more) advance();
      ++g;
      st = st_next;
    };
    // Every slice of a step before the last has its look-ahead slice inside
    // the sweep (when a step has at least kAhead slices): no conditions.
    if (nk >= kAhead && step + 1 < n_steps) {
      slice(true, true);
      for (int kt = 1; kt < nk; ++kt) slice(false, true);
    } else {
      slice(true, false);
      for (int kt = 1; kt < nk; ++kt) slice(false, false);
    }
    const int h0 = h_first + step * h_stride;
    epi(acc, h0, min(h_limit, h0 + kRows));
  }
}

}  // namespace ring

// Sampled group maxima with the ring core (the same scores as the filter
// kernel): block (tile, y) runs samples y * spb .. of the sample list,
// sample s being step s * sample_every; every sampled step is whole.
template <int WQ>
__global__ void __launch_bounds__(ring::Shape<WQ>::kThreads, 2) threshold_sample_ring_kernel(
    EmbView queries, int Q, EmbView hist, int N, int d,
    int sample_every, int n_samples, int spb, float* __restrict__ gm) {
  using S = ring::Shape<WQ>;
  __shared__ __align__(16) char lds[S::kStages * S::kStageBytes];
  const int q0 = blockIdx.x * S::kBQ;
  const int s0 = blockIdx.y * spb;
  const int n_steps = min(spb, n_samples - s0);
  const int lane = (int)lane_id();
  const int w = threadIdx.x / kWave;
  const int wh = w / WQ, wq = w % WQ;
  const int l32 = lane & 31, half = lane >> 5;
  const int stride = sample_every * kStepRows;
  // Sampled steps are whole (256 rows inside the store): no row masking.
  auto epi = [&](floatx16 (&acc)[4][2], int h0, int) {
    const int s = h0 / stride;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int q = q0 + 64 * wq + 32 * t + l32;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float m = acc[u][t][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) m = fmaxf(m, acc[u][t][v]);
        if (q < Q) gm[((size_t)q * n_samples + s) * 16 + wh * 8 + half * 4 + u] = m;
      }
    }
  };
  ring::sweep<WQ>(hist, N, s0 * stride, stride, n_steps, N, queries, Q, q0, d, lds, epi);
}

// Filter kernel: every score >= theta0[q] is written as a key to the
// segment [q][chunk][0..seg_cap) (position from an LDS counter); the true
// count goes to seg_count[q][chunk] even when the segment overflows. With a
// spill array (many small segments) the keys past a full segment go to the
// query's spill[q][0..spill_cap): a chunk whose rows are alike fills its
// segment without sending the query to the exact path.
//
// A kernel without spill array is an instance of its own: with the spill code
// and the threshold that it changes in it, the largest batches, which have
// none, took 1.3% more (28.36 against 28.74 ms at 16,384 x 1M x 1,024).
//
// kAllRows: a store too small for a pre-pass, no threshold, every row of a chunk a
// candidate. Row h of the chunk goes to place h - h_begin of its segment, four
// keys to two stores. Found and picked one by one, 16,000 queries against 2,000
// rows (d = 384) took 565 us a predict, so 243; 60,000 against 1,000 1,194, 520.
enum FilterMode { kSegments, kSpill, kAllRows };
template <int WQ, FilterMode kMode>
__global__ void __launch_bounds__(ring::Shape<WQ>::kThreads, 2) sim_filter_kernel(
    EmbView queries, int Q, EmbView hist, int N, int d,
    int chunk_rows, int n_chunks, int q_tiles, int q_sub, const float* __restrict__ theta0,
    int seg_cap, uint64_t* __restrict__ seg, int* __restrict__ seg_count, int spill_cap,
    uint64_t* __restrict__ spill, int* __restrict__ spill_count, uint32_t* __restrict__ flag_word) {
  using S = ring::Shape<WQ>;
  constexpr bool kAll = kMode == kAllRows;
  __shared__ __align__(16) char lds[S::kStages * S::kStageBytes];
  if (blockIdx.x == 0 && threadIdx.x == 0) *flag_word = 0u;     // set again by the select if it flags a query
  __shared__ int cnt[S::kBQ];
  // Workgroup b runs on XCD b % 8. The (query tile, chunk) pairs are listed in
  // blocks of q_sub tiles, chunk by chunk within a block, and XCD x takes the
  // x-th eighth of the list: the tiles that it works on at a time stay in its
  // L2 while the chunks stream through.
  const int n_pairs = q_tiles * n_chunks;
  const int pair = (int)(blockIdx.x & 7) * ((n_pairs + 7) / 8) + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= (n_pairs + 7) / 8 || pair >= n_pairs) return;
  const int block = pair / (q_sub * n_chunks), r = pair % (q_sub * n_chunks);
  const int in_block = min(q_sub, q_tiles - block * q_sub);
  const int qt = block * q_sub + r % in_block, chunk = r / in_block;
  const int tid = threadIdx.x;
  const int lane = (int)lane_id();
  const int w = tid / kWave;
  const int wh = w / WQ, wq = w % WQ;
  const int l32 = lane & 31, half = lane >> 5;
  const int q0 = qt * S::kBQ;
  const int h_begin = chunk * chunk_rows;
  const int h_end = min(N, h_begin + chunk_rows);
  if (tid < S::kBQ) cnt[tid] = 0;
  float thr[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int q = q0 + 64 * wq + 32 * t + l32;
    thr[t] = !kAll && q < Q ? float_below(theta0[q]) : __builtin_inff();
  }
  // Score acc[u][t][v] of this lane is row h0 + 128 wh + 4 half + r(i) for
  // bit i = 16 u + v, r(i) = 32 (i / 16) + 8 ((i / 4) % 4) + i % 4.
  auto epi_all = [&](floatx16 (&acc)[4][2], int h0, int step_end) {
    const int hl = h0 + 128 * wh + 4 * half;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int q = q0 + 64 * wq + 32 * t + l32;
      if (q >= Q) continue;
      uint64_t* dst = seg + ((size_t)q * n_chunks + chunk) * seg_cap;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
          const int h = hl + 32 * u + 2 * v, j = h - h_begin;      // rows h .. h + 3
          // A quad that the chunk's end cuts is written whole: its segment is the
          // chunk's own, a multiple of four keys, and the count leaves the rest out.
          if (h < step_end && j < seg_cap) {
            ulonglong2* to = reinterpret_cast<ulonglong2*>(dst + j);
            to[0] = make_ulonglong2(make_key(acc[u][t][v], (uint32_t)h), make_key(acc[u][t][v + 1], (uint32_t)h + 1u));
            to[1] = make_ulonglong2(make_key(acc[u][t][v + 2], (uint32_t)h + 2u),
                                    make_key(acc[u][t][v + 3], (uint32_t)h + 3u));
          }
        }
    }
  };
  auto epi = [&](floatx16 (&acc)[4][2], int h0, int step_end) {
    const int lim = step_end - h0 - 128 * wh - 4 * half;     // r(i) < lim: row inside the step
    const int hl = h0 + 128 * wh + 4 * half;
    // Rows inside the step: all of them but in a sweep's last, partial step,
    // where r(i) grows with i, so they are the lowest bits (bits 4g..4g+3 are
    // rows 8g..8g+3, hence the count below).
    uint64_t in_step = ~0ull;
    if (step_end - h0 < kStepRows) {
      const int c = min(max(lim, 0), 128);
      const int n_in = 4 * (c >> 3) + min(c & 7, 4);
      in_step = n_in >= 64 ? ~0ull : (1ull << n_in) - 1ull;
    }
    // The value of bit f (0..15) of a tile: a select tree on the bits of f, as
    // bitwise selects under all-ones / all-zeros masks (one v_bfi each). The
    // masks are opaque to the compiler, which would otherwise fold the tree
    // into a dynamically indexed array and send it through memory.
    auto pick = [](const floatx16& tv, int f) {
      uint32_t sel[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        sel[k] = 0u - (uint32_t)((f >> k) & 1);
        asm volatile("" : "+v"(sel[k]));
      }
      auto bfi = [](uint32_t mask, uint32_t hi, uint32_t lo) { return (hi & mask) | (lo & ~mask); };
      uint32_t a[8], b4[4], c[2];
#pragma unroll
      for (int v = 0; v < 8; ++v) a[v] = bfi(sel[0], __float_as_uint(tv[2 * v + 1]), __float_as_uint(tv[2 * v]));
#pragma unroll
      for (int v = 0; v < 4; ++v) b4[v] = bfi(sel[1], a[2 * v + 1], a[2 * v]);
#pragma unroll
      for (int v = 0; v < 2; ++v) c[v] = bfi(sel[2], b4[2 * v + 1], b4[2 * v]);
      return __uint_as_float(bfi(sel[3], c[1], c[0]));
    };
    // A lane's survivors past their segment's capacity (rare): one device atomic
    // for their places in the spill array. Once that is full the query goes to
    // the exact path whatever else is found, and the lane takes no more of it:
    // with an atomic and a pick for every key, 50,000 equal rows of 100,000 took
    // 300 queries (k = 128, d = 384) 2.3 ms of this kernel against 0.1 without
    // them.
    auto spill_column = [&](int t, uint64_t m, int base) {
      const int q = q0 + 64 * wq + 32 * t + l32;                       // a lane with a survivor has q < Q
      const int kept = min(max(seg_cap - base, 0), __popcll(m));       // of its survivors, in the segment
      const int n = __popcll(m) - kept;
      int e0 = spill_cap;
      if (n > 0) {
        e0 = atomicAdd(&spill_count[q], n);
        if (e0 + n > spill_cap) {
          thr[t] = __builtin_inff();
          e0 = min(e0, spill_cap);                                     // and no overflow of e below
        }
      }
      if (!__any(e0 < spill_cap)) return;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint32_t bits = (uint32_t)(m >> (16 * u)) & 0xffffu;
        while (__any(bits != 0)) {
          const int v = (__ffs(bits) - 1) & 15;
          const float sv = pick(acc[u][t], v);
          if (bits != 0) {
            const int i = 16 * u + v;
            const int e = e0 - kept + __popcll(m & ((1ull << i) - 1ull));
            if (e >= e0 && e < spill_cap)
              spill[(size_t)q * spill_cap + e] = make_key(sv, (uint32_t)(hl + 32 * u + 8 * (v >> 2) + (v & 3)));
            bits &= bits - 1u;
          }
        }
      }
    };
    // Column t's survivors are written one column later, so that its LDS
    // atomic (the segment position) is in flight during the next column's
    // compare. Per tile, a lane's first survivor is picked from the registers;
    // a lane with two or more survivors in one tile (rare) picks the rest one
    // by one.
    uint64_t m_prev = 0;
    int base_prev = 0;
    uint32_t f_prev = 0;
    float fv_prev[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto write_column = [&](int t, uint64_t m, int base, uint32_t fidx, const float (&fv)[4]) {
      const int ql = 64 * wq + 32 * t + l32;
      uint64_t* dst = seg + ((size_t)(q0 + ql) * n_chunks + chunk) * seg_cap;
      uint64_t rest = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t bits = (uint32_t)(m >> (16 * u)) & 0xffffu;
        if (bits != 0) {
          const int f = (int)((fidx >> (4 * u)) & 15u);
          const int i = 16 * u + f;
          const int j = base + __popcll(m & ((1ull << i) - 1ull));     // rank among the lane's survivors
          if (j < seg_cap) dst[j] = make_key(fv[u], (uint32_t)(hl + 32 * u + 8 * (f >> 2) + (f & 3)));
          rest |= (uint64_t)(bits & (bits - 1u)) << (16 * u);
        }
      }
      if (kMode == kSpill && __any(m != 0 && base + __popcll(m) > seg_cap)) spill_column(t, m, base);
      if (!__any(rest != 0)) return;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint32_t bits = (uint32_t)(rest >> (16 * u)) & 0xffffu;
        while (__any(bits != 0)) {
          const int v = (__ffs(bits) - 1) & 15;
          const float sv = pick(acc[u][t], v);
          if (bits != 0) {
            const int i = 16 * u + v;
            const int j = base + __popcll(m & ((1ull << i) - 1ull));
            if (j < seg_cap) dst[j] = make_key(sv, (uint32_t)(hl + 32 * u + 8 * (v >> 2) + (v & 3)));
            bits &= bits - 1u;
          }
        }
      }
    };
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      // Bit v of mk[u] = [acc[u][t][v] > thr]: the sign of thr - s, shifted
      // in with one funnel shift (no compare, so no serialisation on VCC).
      // For finite scores the sign of the rounded difference is exact: -0
      // only arises from a negative difference.
      uint32_t mk[4] = {0u, 0u, 0u, 0u};
      float fv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      uint32_t fidx = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint32_t sg[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) sg[v] = __float_as_uint(thr[t] - acc[u][t][v]);
#pragma unroll
        for (int v = 15; v >= 0; --v) mk[u] = __builtin_amdgcn_alignbit(mk[u], sg[v], 31);
        mk[u] &= (uint32_t)(in_step >> (16 * u)) & 0xffffu;
        if (__any(mk[u] != 0)) {
          const int f = (__ffs(mk[u]) - 1) & 15;
          fv[u] = pick(acc[u][t], f);
          fidx |= (uint32_t)f << (4 * u);
        }
      }
      const uint32_t lo = mk[0] | (mk[1] << 16), hi = mk[2] | (mk[3] << 16);
      const uint64_t m = ((uint64_t)hi << 32) | lo;
      const int ql = 64 * wq + 32 * t + l32;
      const int base = m != 0 ? atomicAdd(&cnt[ql], __popcll(m)) : 0;
      if (t > 0 && __any(m_prev != 0)) write_column(t - 1, m_prev, base_prev, f_prev, fv_prev);
      m_prev = m;
      base_prev = base;
      f_prev = fidx;
#pragma unroll
      for (int u = 0; u < 4; ++u) fv_prev[u] = fv[u];
    }
    if (__any(m_prev != 0)) write_column(1, m_prev, base_prev, f_prev, fv_prev);
  };
  const int n_steps = (h_end - h_begin + kStepRows - 1) / kStepRows;
  if constexpr (kAll) {
    ring::sweep<WQ>(hist, N, h_begin, kStepRows, n_steps, h_end, queries, Q, q0, d, lds, epi_all);
  } else {
    ring::sweep<WQ>(hist, N, h_begin, kStepRows, n_steps, h_end, queries, Q, q0, d, lds, epi);
    __syncthreads();
  }
  if (tid < S::kBQ && q0 + tid < Q)
    seg_count[(size_t)(q0 + tid) * n_chunks + chunk] = kAll ? h_end - h_begin : cnt[tid];
}

template <int NQT, int KL>
hipError_t launch_lists(EmbView queries, int Q, EmbView hist, int N, int d, int k,
                        const SimTopkPlan& p, const float* theta0, const Flagged* only_flagged,
                        uint64_t* partial, hipStream_t stream) {
  LaunchScope scope(only_flagged ? "sim_topk_fallback" : "sim_topk", stream);
  // The fallback runs as one round of workgroups (one per CU) that loop over
  // the tiles, and return at once when no query of the call was flagged.
  const int tiles = p.q_tiles * p.n_chunks;
  if (only_flagged)
    hipLaunchKernelGGL((sim_topk_kernel<NQT, KL, true>), dim3(std::min(tiles, 256)), dim3(kThreads), 0, stream, queries,
                       Q, hist, N, d, k, p.chunk_rows, p.n_chunks, p.q_tiles, theta0, only_flagged->flags,
                       only_flagged->word, partial);
  else
    hipLaunchKernelGGL((sim_topk_kernel<NQT, KL, false>), dim3(tiles), dim3(kThreads), 0, stream, queries, Q, hist, N, d,
                       k, p.chunk_rows, p.n_chunks, p.q_tiles, theta0, nullptr, nullptr, partial);
  return hipGetLastError();
}

// Which kernel scores the sampled steps: each search path samples with the
// arithmetic of its own search, so the sampled scores are the search's own.
enum class Sampler { ring, list, stream };

// Threshold floor for tests of the exact fallback (sage_debug_theta_floor):
// theta0 = max(theta0, floor) before the search.
__global__ void theta_floor_kernel(float* __restrict__ theta0, int Q, float floor) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < Q) theta0[q] = fmaxf(theta0[q], floor);
}

hipError_t launch_theta(EmbView queries, int Q, EmbView hist, int N, int d, int k,
                        const SimTopkPlan& p, int q_tiles, Sampler sampler, float* gm, float* theta0,
                        int* clear, hipStream_t stream) {
  {
    LaunchScope scope("threshold_sample", stream);
    const dim3 grid(q_tiles, p.n_samples);
    if (sampler == Sampler::stream) {
      const hipError_t e = launch_stream_sample(queries, Q, hist, N, d, p.sample_every, p.n_samples, gm, stream);
      if (e != hipSuccess) return e;
    } else if (sampler == Sampler::ring) {
      const int spb = p.f_spb;
      const dim3 rgrid(q_tiles, (p.n_samples + spb - 1) / spb);
      if (p.f_tile == 128)
        hipLaunchKernelGGL(threshold_sample_ring_kernel<2>, rgrid, dim3(ring::Shape<2>::kThreads), 0, stream,
                           queries, Q, hist, N, d, p.sample_every, p.n_samples, spb, gm);
      else
        hipLaunchKernelGGL(threshold_sample_ring_kernel<4>, rgrid, dim3(ring::Shape<4>::kThreads), 0, stream,
                           queries, Q, hist, N, d, p.sample_every, p.n_samples, spb, gm);
    } else if (p.list_len == 128) {              // the same core as sim_topk_kernel<2, 128>
      hipLaunchKernelGGL((threshold_sample_kernel<2>), grid, dim3(kThreads), 0, stream, queries, Q,
                         hist, N, d, p.sample_every, p.n_samples, gm);
    } else {                                     // the same core as sim_topk_kernel<1, 256>
      hipLaunchKernelGGL((threshold_sample_kernel<1>), grid, dim3(kThreads), 0, stream, queries, Q,
                         hist, N, d, p.sample_every, p.n_samples, gm);
    }
  }
  const int m = p.n_samples * 16;
  LaunchScope scope("threshold_select", stream);
  if (Q < 512) {                                       // one 16-wave workgroup per query
    if (m <= 2 * 16 * kWave)
      hipLaunchKernelGGL((threshold_select_kernel<2, 16>), dim3(Q), dim3(1024), 0, stream, gm, Q, m, k, theta0, clear);
    else
      hipLaunchKernelGGL((threshold_select_kernel<8, 16>), dim3(Q), dim3(1024), 0, stream, gm, Q, m, k, theta0, clear);
  } else {                                             // four queries (wavefronts) per workgroup
    const dim3 grid((Q + 3) / 4);
    if (m <= 16 * kWave)
      hipLaunchKernelGGL((threshold_select_kernel<16, 1>), grid, dim3(256), 0, stream, gm, Q, m, k, theta0, clear);
    else if (m <= 32 * kWave)
      hipLaunchKernelGGL((threshold_select_kernel<32, 1>), grid, dim3(256), 0, stream, gm, Q, m, k, theta0, clear);
    else if (m <= 64 * kWave)
      hipLaunchKernelGGL((threshold_select_kernel<64, 1>), grid, dim3(256), 0, stream, gm, Q, m, k, theta0, clear);
    else
      hipLaunchKernelGGL((threshold_select_kernel<128, 1>), grid, dim3(256), 0, stream, gm, Q, m, k, theta0, clear);
  }
  const float floor = debug_theta_floor();
  if (sampler != Sampler::list && floor > -__builtin_inff())   // only the paths with a guarded fallback
    hipLaunchKernelGGL(theta_floor_kernel, dim3((Q + 255) / 256), dim3(256), 0, stream, theta0, Q, floor);
  return hipGetLastError();
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

void chunking(int q_tiles, int N, int target_blocks, int max_chunks, int* chunk_rows, int* n_chunks) {
  const long steps = ((long)N + kStepRows - 1) / kStepRows;
  long want = ((long)target_blocks + q_tiles - 1) / (long)(q_tiles > 0 ? q_tiles : 1);
  if (want >= 8) want = (want + 7) / 8 * 8;            // whole chunks per XCD
  if (want < 1) want = 1;
  if (want > max_chunks) want = max_chunks;
  if (want > steps) want = steps;
  long rows = ((long)N + want - 1) / want;
  rows = (rows + kStepRows - 1) / kStepRows * kStepRows;
  *chunk_rows = (int)rows;
  *n_chunks = (int)(((long)N + rows - 1) / rows);
}

// Chunks of the filter kernel: the number of 256-row steps per workgroup that
// gives the shortest makespan of q_tiles * n_chunks workgroups on `slots`,
// each costing its steps and about half a step for its start and end. Chunk
// counts are multiples of 8 (whole chunks per XCD) up to what the select can
// take: 512 with a spill array for segments that fill up, else 64.
void filter_chunking(int q_tiles, int N, int slots, bool spill, int* chunk_rows, int* n_chunks) {
  const long steps = ((long)N + kStepRows - 1) / kStepRows;
  long best = 1;
  double best_cost = -1.0;
  const long most = !spill ? 64 : (q_tiles == 1 ? 512 : (q_tiles <= 8 ? 256 : 64));
  for (long want = 8; want <= most; want += 8) {
    const long per = (steps + want - 1) / want, chunks = (steps + per - 1) / per;
    const long rounds = (chunks * q_tiles + slots - 1) / slots;
    const double cost = rounds * per * (1.0 + 0.05 / rounds) + 0.5 * rounds;
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = per; }
  }
  *chunk_rows = (int)(best * kStepRows);
  *n_chunks = (int)((steps + best - 1) / best);
}

// Workspace layout (byte offsets) of a plan whose path is chosen.
void plan_workspace(SimTopkPlan* p, int Q, int L) {
  size_t o = 0;
  // One region for what is dead before the next of it is written: the sampled
  // maxima (read by the threshold select), the candidates (by the candidate
  // select) and the exact lists (the fallback runs last).
  const int groups = merge_groups(Q, p->n_chunks, L);
  p->off_partial = o;
  p->off_merge = align256(p->off_partial + (size_t)Q * p->n_chunks * L * sizeof(uint64_t));
  const size_t lists_end = align256(p->off_merge + (groups > 1 ? (size_t)Q * groups * L * sizeof(uint64_t) : 0));
  if (p->fast) {
    p->off_seg = o;    o = align256(o + (size_t)Q * p->f_n_chunks * p->seg_cap * sizeof(uint64_t));
    p->off_spill = o;  o = align256(o + (size_t)Q * p->spill_cap * sizeof(uint64_t));
  }
  if (p->stream) { p->off_cand = o; o = align256(o + (size_t)Q * p->s_cap * sizeof(uint64_t)); }
  p->off_gm = 0;
  o = std::max(std::max(o, lists_end), align256((size_t)Q * p->n_samples * 16 * sizeof(float)));
  p->off_theta = o;   o = align256(o + (size_t)Q * sizeof(float));
  if (p->fast) {
    p->off_segcnt = o; o = align256(o + (size_t)Q * p->f_n_chunks * sizeof(int));
    p->off_spillcnt = o; o = align256(o + (p->spill_cap > 0 ? (size_t)Q * sizeof(int) : 0));
  }
  if (p->stream) { p->off_ccount = o; o = align256(o + (size_t)Q * sizeof(int)); }
  if (p->fast || p->stream) {
    p->off_flags = o;  o = align256(o + (size_t)Q * sizeof(int));
    p->off_flag_word = o; o = align256(o + sizeof(uint32_t));
  }
  p->total_bytes = o;
}

bool dense_takes(int Q, int N, int d) {
  return Q <= kDenseMaxQ && N <= kDenseMaxRows && d <= kDenseMaxD && (long)Q * N <= kDenseMaxScores;
}
// Whether writing every score out is the faster search, from its and the
// filtered search's times (us, measured at k = 64 over 17 to 1,024 queries, 64
// to 32,768 rows and d = 384 to 8,192, both layouts). Up to 256 queries it is,
// or is at least no slower than any search was before it; for k > 64 the other
// one is mostly the exact lists, two to three times slower but for a single tile
// of rows and k > 128, whose lists hold all of them (dense / lists, k = 256:
// 1,024 x 50 x 128 67 / 38, x 2,048 72 / 62; 600 x 100 x 128 62 / 57; 600 x 10 x
// 2,048 46 / 55). Past that its select
// takes a workgroup of 16 waves per query, about 36 ns each, and every 32 x 32
// tile fetches its own operands: 1.6e14 products a second, and 0.7e14 where
// rows lie d apart, so that a load touches twice as many cache lines. The
// filtered search is one round of tiles at these sizes, its time the latency of
// d / 32 slices, twice that with a pre-pass. Dense / filtered, panels and rows:
// 1,024 x 5,000 x 768 68 / 62 and 91 / 63, x 8,192 294 / 190 and 544 / 192;
// 512 x 10,000 x 768 52 / 59 and 75 / 60; 512 x 5,000 x 384 36 / 54 and 43 / 54;
// 1,024 x 64 x 384 45 / 28.
bool dense_pays(int Q, int N, int d, int k, bool sampled, bool panels) {
  if (!dense_takes(Q, N, d)) return false;
  if (Q <= 256) return true;
  if (k > 64) return !(k > 128 && N <= 128 && 0.06 * Q > 20.0 + d / 64.0);
  const double dense = 4.0 + 0.036 * Q + (double)Q * N * d / (panels ? 1.6e8 : 0.7e8);
  const double filtered = sampled ? 35.0 + d / 30.0 : std::min(48.0, 20.0 + 0.017 * N) + d / 60.0;
  return dense <= filtered;
}

}  // namespace

SimTopkPlan plan_sim_topk(int Q, int N, int d, int k, size_t limit, PlanFor layout) {
  SimTopkPlan p{};
  int L = 64;
  while (L < k) L <<= 1;
  p.list_len = L;
  p.q_tile = L == 64 ? 128 : (L == 128 ? 64 : 32);
  p.q_tiles = (Q + p.q_tile - 1) / p.q_tile;
  chunking(p.q_tiles, N, 1024, 1 << 20, &p.chunk_rows, &p.n_chunks);
  // Threshold pre-pass: every SR-th step, >= 4k group maxima, at most 8192.
  // SR <= 16: every candidate above theta0 is written out, so a tighter bound
  // pays for the larger sample. The sample costs about Q N d / SR and the
  // candidates about Q k SR, so the best SR grows with the square root of
  // N d / k: from N d = 2^29 on (1M keys of d = 1024) k <= 64 samples every
  // 32nd step. For k > 64, decisions of 2,048 queries against 500,000 x 768 at
  // SR 8 / 16 / 32: k = 128 1,471 / 1,421 / 1,436 us, k = 256 1,528 / 1,501 /
  // 1,678 us.
  // Only whole steps are sampled.
  const long steps = (long)N / kStepRows;
  if (steps * 16 >= 8L * k) {
    // The stream path (few queries) reads the whole store anyway and pays for
    // candidates only in its select: it samples every 128th step at most
    // (streaming workload: pre-pass 44 -> 16 us, select 16 -> 25 us, call -1.5%).
    const bool wide = Q > kStreamMaxQ && (long)N * d >= (1L << 29);
    const bool few = Q <= kStreamMaxQ && d <= kStreamMaxD && k <= 256;     // the stream path's shapes
    const long sr_max = few ? 128 : (L == 64 && wide ? 32 : 16);
    long sr = steps * 16 / (4L * k);
    if (sr > sr_max) sr = sr_max;
    if (sr < 1) sr = 1;
    while ((steps + sr - 1) / sr > 512) ++sr;
    // A batch of few 256-query tiles leaves CUs idle while it samples: twice
    // the samples cost nothing there, and halve the candidates, while they
    // still fit one round of workgroups and the threshold select's smallest
    // kernel (1,024 maxima; 2,048 with 16 waves per query).
    if (Q > 128) {
      const long tiles = (Q + 255) / 256, most = std::min(256 / tiles, Q >= 512 ? 64L : 128L);
      while (sr > 1 && (steps + sr / 2 - 1) / (sr / 2) <= most) sr /= 2;
    }
    p.sample_every = (int)sr;
    p.n_samples = (int)((steps + sr - 1) / sr);
  }
  // Small store and batch: every score written out (up to 20 MB of them).
  const size_t scores = align256((size_t)Q * ((N + 31) / 32 * 32) * sizeof(float));
  auto dense = [&]() {
    SimTopkPlan p{};
    p.dense = true;
    p.dense_ld = (N + 31) / 32 * 32;
    p.total_bytes = scores;
    return p;
  };
  if (dense_pays(Q, N, d, k, p.n_samples > 0, false)) return dense();
  // Where it pays on panels only, the layout decides: the workspace holds either
  // search, and a word in it says which one ran.
  const bool by_layout = dense_pays(Q, N, d, k, p.n_samples > 0, true);
  // Few queries against a large store: the stream path (one pass over the
  // store, bound by HBM), given a threshold pre-pass.
  p.stream = Q <= kStreamMaxQ && d <= kStreamMaxD && k <= 256 && p.n_samples > 0;
  // Filtered path: segments of 8192 keys per query in all. k > 64 needs the
  // pre-pass (all rows of a store too small for one would be candidates); the
  // exact lists, which it replaces there, take 4,620 against 1,421 us at
  // 2,048 x 500,000 x 768 and k = 128, 7,803 against 1,501 us at k = 256, and
  // 157 against 80 us at 200 x 20,000 x 768 and k = 128.
  p.fast = !p.stream && (L == 64 || p.n_samples > 0);
  if (p.fast) {
    // Up to 128 queries the search is one pass over the store, bound by HBM:
    // a 128-query tile halves the work done for padding, and two of its
    // workgroups share a CU.
    p.f_tile = Q <= 128 ? 128 : 256;
    p.f_q_tiles = (Q + p.f_tile - 1) / p.f_tile;
    const int slots = p.f_tile == 128 ? 512 : 256;   // workgroups the chip holds at a time
    // samples per sampling block: about one block per slot (with 256 query
    // tiles and more, one block per tile)
    p.f_spb = 1;
    while (p.f_spb < p.n_samples && (long)p.f_q_tiles * ((p.n_samples + 2 * p.f_spb - 1) / (2 * p.f_spb)) >= 256)
      p.f_spb *= 2;
    filter_chunking(p.f_q_tiles, N, slots, p.n_samples > 0, &p.f_chunk_rows, &p.f_n_chunks);
    // Query tiles that an XCD works on at a time: as many (all of them, or a
    // power of two) as take at most 3 MiB of its 4 MiB L2. On 64 tiles of
    // 512 KiB, 4 at a time against all 64 against one chunk, same box:
    // 30.45 -> 29.65 ms (2 at a time 30.25).
    const long fit = std::max(1L, (3L << 20) / ((long)p.f_tile * d * 2));
    p.f_q_sub = p.f_q_tiles;
    if (p.f_q_tiles > fit)
      for (p.f_q_sub = 1; p.f_q_sub * 2 <= fit; p.f_q_sub *= 2) {}
    p.seg_cap = 1;                                   // power of two, n_chunks * cap <= 8192
    while (p.seg_cap * 2 * p.f_n_chunks <= 8192) p.seg_cap *= 2;
    // Segments of fewer than 128 keys (more than 64 chunks) fill easily where
    // a chunk's rows are alike: the rest goes to the query's spill array.
    // So do those of k > 64, whose candidates are more.
    p.spill_cap = p.f_n_chunks > 64 || L > 64 ? 4096 : 0;
  }
  // Stream path: about k * SR keys beat theta0 per query; the array holds four
  // times that.
  if (p.stream) {
    long rows = ((long)N + 511) / 512;                   // about two workgroups per CU
    rows = (rows + 63) / 64 * 64;
    p.s_chunk_rows = (int)rows;
    p.s_cap = 4096;
    while (p.s_cap < 4L * k * p.sample_every) p.s_cap *= 2;
  }
  plan_workspace(&p, Q, L);
  if (by_layout && p.total_bytes + scores <= limit) {  // then k <= 64, on the filtered path
    p.by_layout = true;
    p.dense = layout == PlanFor::panels;
    p.dense_ld = (N + 31) / 32 * 32;
    p.off_scores = p.total_bytes;
    p.total_bytes += scores;
    return p;
  }
  if (scores <= limit && ((by_layout && layout == PlanFor::panels) ||
                          (p.total_bytes > limit && dense_takes(Q, N, d)))) return dense();
  // The exact lists alone take less. They are three times slower (figures
  // above), so a search of k > 64 keeps to them only where the scratch is
  // given and holds them and not the candidates.
  if (p.fast && L > 64 && p.total_bytes > limit) {
    SimTopkPlan lists = p;
    lists.fast = false;
    plan_workspace(&lists, Q, L);
    if (lists.total_bytes <= limit) return lists;
  }
  return p;
}

hipError_t launch_neighbours(EmbView queries, int Q, EmbView hist, int N, int d, int k,
                             const SimTopkPlan& p, void* workspace, int32_t* ids, float* sims,
                             const DenseHist& hist_part, hipStream_t stream) {
  if (Q == 0) return hipSuccess;
  char* ws = static_cast<char*>(workspace);
  if (p.dense)
    return launch_dense(queries, Q, hist, N, d, k, p.dense_ld, reinterpret_cast<float*>(ws + p.off_scores),
                        p.by_layout ? reinterpret_cast<uint32_t*>(ws + p.off_flag_word) : nullptr, ids, sims,
                        hist_part, stream);
  uint64_t* partial = reinterpret_cast<uint64_t*>(ws + p.off_partial);
  uint64_t* merge_lists = reinterpret_cast<uint64_t*>(ws + p.off_merge);
  float* gm = reinterpret_cast<float*>(ws + p.off_gm);
  float* theta0 = reinterpret_cast<float*>(ws + p.off_theta);
  hipError_t e;
  if (p.fast) {
    uint64_t* spill = reinterpret_cast<uint64_t*>(ws + p.off_spill);
    int* spillcnt = p.spill_cap > 0 ? reinterpret_cast<int*>(ws + p.off_spillcnt) : nullptr;
    if (p.n_samples > 0) {                             // a spill array comes with a pre-pass, which clears its counts
      e = launch_theta(queries, Q, hist, N, d, k, p, p.f_q_tiles, Sampler::ring, gm, theta0, spillcnt, stream);
      if (e != hipSuccess) return e;
    }
    uint64_t* seg = reinterpret_cast<uint64_t*>(ws + p.off_seg);
    int* segcnt = reinterpret_cast<int*>(ws + p.off_segcnt);
    const Flagged fl{reinterpret_cast<int*>(ws + p.off_flags), reinterpret_cast<uint32_t*>(ws + p.off_flag_word)};
    {
      LaunchScope scope("sim_topk", stream);
      const dim3 grid((p.f_q_tiles * p.f_n_chunks + 7) / 8 * 8);
#define SAGE_FILTER(WQ, MODE)                                                                                      \
  hipLaunchKernelGGL((sim_filter_kernel<WQ, MODE>), grid, dim3(ring::Shape<WQ>::kThreads), 0, stream, queries, Q,   \
                     hist, N, d, p.f_chunk_rows, p.f_n_chunks, p.f_q_tiles, p.f_q_sub, theta0, p.seg_cap, seg, segcnt, \
                     p.spill_cap, spill, spillcnt, fl.word)
      if (p.n_samples == 0) {
        if (p.f_tile == 128) SAGE_FILTER(2, kAllRows); else SAGE_FILTER(4, kAllRows);
      } else if (p.spill_cap > 0) {
        if (p.f_tile == 128) SAGE_FILTER(2, kSpill); else SAGE_FILTER(4, kSpill);
      } else {
        if (p.f_tile == 128) SAGE_FILTER(2, kSegments); else SAGE_FILTER(4, kSegments);
      }
#undef SAGE_FILTER
    }
    const Candidates cand{seg, segcnt, p.f_n_chunks, p.seg_cap, spill, spillcnt, p.spill_cap};
    e = launch_select(cand, Q, k, min(k, N), fl, ids, sims, stream);
    if (e != hipSuccess) return e;
    // Exact fallback for queries whose candidates overflowed (no work otherwise).
    // Its scores are the filter kernel's, bit for bit, so theta0 bounds them too.
    const float* th = p.n_samples > 0 ? theta0 : nullptr;
    if (p.list_len == 64) e = launch_lists<4, 64>(queries, Q, hist, N, d, k, p, th, &fl, partial, stream);
    else if (p.list_len == 128) e = launch_lists<2, 128>(queries, Q, hist, N, d, k, p, th, &fl, partial, stream);
    else e = launch_lists<1, 256>(queries, Q, hist, N, d, k, p, th, &fl, partial, stream);
    if (e != hipSuccess) return e;
    return launch_topk_merge(partial, Q, p.n_chunks, p.list_len, k, &fl, merge_lists, ids, sims, stream);
  }
  if (p.stream) {
    uint64_t* cand = reinterpret_cast<uint64_t*>(ws + p.off_cand);
    int* ccount = reinterpret_cast<int*>(ws + p.off_ccount);
    const Flagged fl{reinterpret_cast<int*>(ws + p.off_flags), reinterpret_cast<uint32_t*>(ws + p.off_flag_word)};
    e = launch_theta(queries, Q, hist, N, d, k, p, 1, Sampler::stream, gm, theta0, ccount, stream);
    if (e != hipSuccess) return e;
    e = launch_stream_search(queries, Q, hist, N, d, p.s_chunk_rows, theta0, p.s_cap, cand, ccount, fl.word, stream);
    if (e != hipSuccess) return e;
    e = launch_select(Candidates{nullptr, nullptr, 0, 0, cand, ccount, p.s_cap}, Q, k, min(k, N), fl, ids, sims, stream);
    if (e != hipSuccess) return e;
    // Exact fallback for queries whose candidates overflowed (no work otherwise);
    // its scores may differ from the stream kernel's in the last bit: no threshold.
    if (p.list_len == 64) e = launch_lists<4, 64>(queries, Q, hist, N, d, k, p, nullptr, &fl, partial, stream);
    else if (p.list_len == 128) e = launch_lists<2, 128>(queries, Q, hist, N, d, k, p, nullptr, &fl, partial, stream);
    else e = launch_lists<1, 256>(queries, Q, hist, N, d, k, p, nullptr, &fl, partial, stream);
    if (e != hipSuccess) return e;
    return launch_topk_merge(partial, Q, p.n_chunks, p.list_len, k, &fl, merge_lists, ids, sims, stream);
  }
  if (p.n_samples > 0) {
    e = launch_theta(queries, Q, hist, N, d, k, p, p.q_tiles, Sampler::list, gm, theta0, nullptr, stream);
    if (e != hipSuccess) return e;
  }
  const float* th = p.n_samples > 0 ? theta0 : nullptr;
  if (p.list_len == 128) e = launch_lists<2, 128>(queries, Q, hist, N, d, k, p, th, nullptr, partial, stream);
  else e = launch_lists<1, 256>(queries, Q, hist, N, d, k, p, th, nullptr, partial, stream);
  if (e != hipSuccess) return e;
  return launch_topk_merge(partial, Q, p.n_chunks, p.list_len, k, nullptr, merge_lists, ids, sims, stream);
}

}  // namespace sage
