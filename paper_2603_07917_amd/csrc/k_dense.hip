// Neighbour search of a small batch against a small store (Sec. 3.1: the
// method's own window holds 10,000 prompts): every score is written out and
// each query selects from its row.
//
// At these sizes the searches with a threshold pre-pass are bound by their
// launches (sample, threshold, search, select, and two for a fallback that
// has nothing to do) and fill a few dozen workgroups. Here two launches do the
// search, with nothing to fall back from.
#include <algorithm>

#include "sage_device.hpp"
#include "sage_hist.hpp"
#include "sage_internal.hpp"
#include "sage_toplist.hpp"

namespace sage {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

// S[q][n] for a tile of 32 queries (blockIdx.y) and 32 kTiles history rows per
// wave: d / 16 chained v_mfma_f32_32x32x16_bf16 from zero in column order,
// which gives the bits of the filtered search. Operands go straight from
// global memory to registers, kPanels 32-column panels in flight: a wave waits
// d / (32 kPanels) times, and there is no barrier.
// A operand: queries; B operand: history rows, so that a store instruction
// writes 32 consecutive scores of a query. Rows and queries past the end are
// read clamped and not stored.
template <int kTiles>
__global__ void __launch_bounds__(256, 2) dense_score_kernel(EmbView queries, int Q, EmbView hist, int N, int d,
                                                             int ld, float* __restrict__ scores) {
  constexpr int kPanels = kTiles == 1 ? 12 : 6;
  const int lane = (int)lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int l32 = lane & 31, half = lane >> 5;
  const int n0 = (int)(blockIdx.x * (blockDim.x / kWave) + w) * (32 * kTiles), q0 = blockIdx.y * 32;
  if (n0 >= N) return;                              // whole waves; no barrier below
  // Uniform panel address plus a per-lane byte offset (below 2^32: d <= kDenseMaxD).
  const uint32_t q_off = ((uint32_t)min(q0 + l32, Q - 1) * (uint32_t)queries.row + 8u * half) * 2u;
  uint32_t h_off[kTiles];
#pragma unroll
  for (int t = 0; t < kTiles; ++t)
    h_off[t] = ((uint32_t)min(n0 + 32 * t + l32, N - 1) * (uint32_t)hist.row + 8u * half) * 2u;
  const int KB = d / 32;
  floatx16 acc[kTiles] = {};
  for (int k0 = 0; k0 < KB; k0 += kPanels) {
    bf16x8 a[kPanels][2], b[kPanels][kTiles][2];
#pragma unroll
    for (int i = 0; i < kPanels; ++i)
      if (k0 + i < KB) {
        const char* qi = reinterpret_cast<const char*>(queries.base + (long long)(k0 + i) * queries.panel);
        const char* hi = reinterpret_cast<const char*>(hist.base + (long long)(k0 + i) * hist.panel);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          a[i][j] = *reinterpret_cast<const bf16x8*>(qi + q_off + 32 * j);
#pragma unroll
          for (int t = 0; t < kTiles; ++t) b[i][t][j] = *reinterpret_cast<const bf16x8*>(hi + h_off[t] + 32 * j);
        }
      }
#pragma unroll
    for (int i = 0; i < kPanels; ++i)
      if (k0 + i < KB) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int t = 0; t < kTiles; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][j], b[i][t][j], acc[t], 0, 0, 0);
      }
  }
#pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    const int n = n0 + 32 * t + l32;
    if (n >= N) continue;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int q = q0 + 8 * (v >> 2) + 4 * half + (v & 3);
      if (q < Q) scores[(size_t)q * ld + n] = acc[t][v];
    }
  }
}

// One workgroup of 16 waves per query; thread t holds scores t, t + 1024, ...
// (at most kPer, in registers). A lower bound T on the k-th best score is the
// k-th largest of disjoint groups' maxima (256 groups of four threads, or each
// thread's own for k > 128), found bit by bit by one wave; about k keys
// (1.15 k at k = 64) reach it. They are gathered in LDS, sorted 64 to a wave
// and merged (as in the candidate select). Where more than the LDS holds reach
// T (equal scores), every wave folds all of its keys instead: slower, exact.
//
// With counts, the neighbours then go through the histogram in place (as in
// the histogram kernel: exact fixed-point weights, so the same bits), which
// saves its launch.
template <int S, int kPer>
__global__ void __launch_bounds__(1024) dense_select_kernel(const float* __restrict__ scores, int N, int ld, int k,
                                                            uint32_t* __restrict__ ran, int32_t* __restrict__ ids,
                                                            float* __restrict__ sims, DenseHist h) {
  constexpr int KL = 64 * S;
  constexpr int W = 16;
  constexpr int kCap = 1024;
  constexpr int kGroups = S <= 2 ? 4 : 16;          // group maxima per lane of the wave that finds T
  __shared__ uint64_t lists[W][KL];
  __shared__ uint64_t pend[W][2 * kWave];
  __shared__ uint64_t cand[kCap];
  __shared__ uint32_t gmax[64 * kGroups];
  __shared__ uint32_t bound;
  __shared__ int n_cand, n_nbr;
  __shared__ uint64_t w_all;
  // Histogram (8-byte words): weights [B], edges [B + 1], then counts [B] (4-byte).
  extern __shared__ __align__(16) unsigned char hist_smem[];
  uint64_t* wsum = reinterpret_cast<uint64_t*>(hist_smem);
  double* edges = reinterpret_cast<double*>(hist_smem) + h.B;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(edges + h.B + 1);
  const int q = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = (int)lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const float* row = scores + (size_t)q * ld;
  // The scores as monotone bits; 0 (below every score's) past the end.
  uint32_t s[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) s[i] = i * 1024 + tid < N ? __float_as_uint(row[i * 1024 + tid]) : 0u;
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    s[i] = i * 1024 + tid < N ? f32_order_bits(__uint_as_float(s[i])) : 0u;
    m = max(m, s[i]);
  }
  if (kGroups == 4) {
    m = max(m, xor_lane_u32<1>(m));
    m = max(m, xor_lane_u32<2>(m));
    if ((lane & 3) == 0) gmax[tid >> 2] = m;
  } else {
    gmax[tid] = m;
  }
  if (tid == 0) {
    n_cand = 0;
    n_nbr = 0;
    w_all = 0;
  }
  for (int b = tid; b <= h.B; b += 1024) {          // no histogram: B = -1
    edges[b] = h.edges[b];
    if (b < h.B) {
      wsum[b] = 0;
      cnt[b] = 0;
    }
  }
  __syncthreads();
  if (w == 0) {
    uint32_t key[kGroups], hi = 0, lo = 0xffffffffu;
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
      key[i] = gmax[i * kWave + lane];
      hi = max(hi, key[i]);
      lo = min(lo, key[i]);
    }
    hi = wave_max_dpp_u32(hi);
    lo = wave_min_dpp_u32(lo);
    // The largest T with at least k maxima >= T (0 when fewer than k groups
    // hold a score); the bits above the first where hi and lo differ are fixed.
    const int top = hi == lo ? -1 : 31 - __clz(hi ^ lo);
    uint32_t T = top < 0 ? hi : hi & ~((2u << top) - 1u);
    for (int bit = top; bit >= 0; --bit) {
      const uint32_t c = T | (1u << bit);
      int n = 0;
#pragma unroll
      for (int i = 0; i < kGroups; ++i) n += __popcll(__ballot(key[i] >= c));
      if (n >= k) T = c;
    }
    if (lane == 0) bound = T;
  }
  __syncthreads();
  const uint32_t T = max(bound, 1u);                // never the 0 of no score
  int mine = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) mine += s[i] >= T ? 1 : 0;
  if (mine > 0) {
    int pos = atomicAdd(&n_cand, mine);
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (s[i] >= T) {
        if (pos < kCap) cand[pos] = ((uint64_t)s[i] << 32) | (uint64_t)~(uint32_t)(i * 1024 + tid);
        ++pos;
      }
  }
  __syncthreads();
  const int n = n_cand;
  TopList<S> top(pend[w]);
  if (n <= kCap) {
    for (int e = w * kWave; e < n; e += W * kWave) top.take(e + lane < n ? cand[e + lane] : kPadKey);
  } else {
    for (int r = tid; r - lane < N; r += 1024) top.take(r < N ? make_key(row[r], (uint32_t)r) : kPadKey);
  }
  top.flush();
  merge_lists<S, W>(top.lv, &lists[0][0], w, n <= kCap ? (n + kWave - 1) / kWave : W);
  if (w == 0) top.write(k, ids + (size_t)q * k, sims + (size_t)q * k);
  else if (q == 0 && tid == 1023 && ran) *ran = kDenseRan;       // here, where no other wave waits for it
  if (h.B < 1) return;
  if (w == 0) {
    int32_t len[S];
    bool in[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      in[s] = 64 * s + lane < k && top.lv[s] != kPadKey;
      len[s] = in[s] ? h.hist_len[key_id(top.lv[s])] : 0;
    }
    uint64_t mine_w = 0;
    int mine_n = 0;
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (in[s]) {
        const int b = length_bin(edges, h.B, len[s]);
        const float sim = key_sim(top.lv[s]);
        atomicAdd(&cnt[b], 1u);
        ++mine_n;
        if (sim >= h.tau) {
          const uint64_t fx = weight_fixed(sim, false);
          atomicAdd(reinterpret_cast<unsigned long long*>(&wsum[b]), (unsigned long long)fx);
          mine_w += fx;
        }
      }
    if (mine_n > 0) {
      atomicAdd(&n_nbr, mine_n);
      atomicAdd(reinterpret_cast<unsigned long long*>(&w_all), (unsigned long long)mine_w);
    }
  }
  __syncthreads();
  const uint64_t wtot = w_all;
  const bool weighted = wtot > 0;
  const double scale = weighted ? 1.0 / (double)wtot : (n_nbr > 0 ? 1.0 / (double)n_nbr : 0.0);
  for (int b = tid; b < h.B; b += 1024) {
    h.counts[(size_t)q * h.B + b] = (int32_t)cnt[b];
    h.mass[(size_t)q * h.B + b] = (float)((weighted ? (double)wsum[b] : (double)cnt[b]) * scale);
  }
}

template <int S>
void launch_dense_select(const float* scores, int Q, int N, int ld, int k, uint32_t* ran, int32_t* ids, float* sims,
                         const DenseHist& h, hipStream_t stream) {
  const size_t lds = h.B > 0 ? (size_t)h.B * 20 + 8 : 0;
  if (N <= 8192)
    hipLaunchKernelGGL((dense_select_kernel<S, 8>), dim3(Q), dim3(1024), lds, stream, scores, N, ld, k, ran, ids,
                       sims, h);
  else if (N <= 16384)
    hipLaunchKernelGGL((dense_select_kernel<S, 16>), dim3(Q), dim3(1024), lds, stream, scores, N, ld, k, ran, ids,
                       sims, h);
  else
    hipLaunchKernelGGL((dense_select_kernel<S, 32>), dim3(Q), dim3(1024), lds, stream, scores, N, ld, k, ran, ids,
                       sims, h);
}
static_assert(kDenseMaxRows == 32 * 1024, "the last case holds the largest store");

}  // namespace

hipError_t launch_dense(EmbView queries, int Q, EmbView hist, int N, int d, int k, int ld, float* scores,
                        uint32_t* ran, int32_t* ids, float* sims, const DenseHist& h, hipStream_t stream) {
  if (Q <= 0 || Q > kDenseMaxQ || N <= 0 || N > kDenseMaxRows || ld < N || k < 1 || k > 256 || d % 32 != 0 ||
      d > kDenseMaxD || h.B > kDenseHistMaxBins) return hipErrorInvalidValue;
  {
    LaunchScope scope("sim_topk", stream);
    // Up to one 32 x 32 tile per SIMD: single-wave workgroups, which spread
    // over more CUs. From two per SIMD on, two tiles per wave share the query
    // operands, a quarter less to read through L2 (128 x 32,768 x 768: decision
    // 50.9 -> 41.1 us, 500 x 10,000 x 768 64.0 -> 55.5, 256 x 8,192 x 384 the same).
    const long tiles = (long)((N + 31) / 32) * ((Q + 31) / 32);
    const unsigned gy = (unsigned)((Q + 31) / 32);
    if (tiles <= 1024)
      hipLaunchKernelGGL(dense_score_kernel<1>, dim3((N + 31) / 32, gy), dim3(kWave), 0, stream, queries, Q, hist, N, d,
                         ld, scores);
    else if (tiles < 2048)
      hipLaunchKernelGGL(dense_score_kernel<1>, dim3((N + 127) / 128, gy), dim3(4 * kWave), 0, stream, queries, Q, hist,
                         N, d, ld, scores);
    else
      hipLaunchKernelGGL(dense_score_kernel<2>, dim3((N + 255) / 256, gy), dim3(4 * kWave), 0, stream, queries, Q, hist,
                         N, d, ld, scores);
  }
  LaunchScope scope(h.B > 0 ? "hist" : "topk_select", stream);   // the histogram ends it, where it is part
  if (k <= 64) launch_dense_select<1>(scores, Q, N, ld, k, ran, ids, sims, h, stream);
  else if (k <= 128) launch_dense_select<2>(scores, Q, N, ld, k, ran, ids, sims, h, stream);
  else launch_dense_select<4>(scores, Q, N, ld, k, ran, ids, sims, h, stream);
  return hipGetLastError();
}

}  // namespace sage
