// Candidate select: each query's k best keys out of the candidates that a
// search wrote for it (the keys at or above its pre-pass threshold).
#include "sage_device.hpp"
#include "sage_internal.hpp"
#include "sage_toplist.hpp"

namespace sage {
namespace {

// W wavefronts per query. Wave w takes the w-th share of the query's segments
// (at most 64; they form one index range, kPre groups of 64 keys in flight)
// and every W-th group of 64 of its spill array. Only keys that beat the
// wave's running (64 S)-th key are gathered in LDS and folded, 64 at a time,
// into its list (S registers per lane). The W lists are then merged pairwise
// in a tree: C_p = max(A_p, B_(KL-1-p)) is bitonic and holds the best of both.
// A query whose candidates overflowed, or that has fewer than min(k, N) of
// them (the pre-pass scores are the search's own, bit for bit, so only a
// raised threshold can cause it), is flagged for the exact fallback and left
// untouched here.
//
// W = 1: four queries per workgroup and no workgroup barrier; one list per
// query means that only about k (1 + ln(n / k)) of n keys are sorted. W > 1
// (few queries): a single wave per query would leave the chip idle and each
// wave bound by the latency of its own loads and folds.
//
// kSeg: the query has segments (else a spill array only).
template <int S, int W, bool kSeg>
__global__ void __launch_bounds__(W == 1 ? 256 : 64 * W) select_kernel(Candidates c, int Q, int k, int need,
                                                                       Flagged fl, int32_t* __restrict__ ids,
                                                                       float* __restrict__ sims) {
  constexpr int KL = 64 * S;
  constexpr int WG = W == 1 ? 4 : W;                  // wavefronts per workgroup
  __shared__ int off_s[WG][kWave];
  __shared__ uint64_t pend[WG][2 * kWave];
  __shared__ uint64_t lists[W == 1 ? 1 : W][W == 1 ? 1 : KL];
  __shared__ int tot_s[W], over_s[W];
  const int lane = (int)lane_id();
  const int wg = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int w = W == 1 ? 0 : wg;
  const int q = W == 1 ? (int)blockIdx.x * 4 + wg : (int)blockIdx.x;
  if (q >= Q) return;                                 // whole wavefronts, only for W = 1
  int* off = off_s[wg];
  // Segment c0 + l (one per lane) starts at off[l] of this wave's index range.
  const int per = (c.n_chunks + W - 1) / W;
  const int c0 = w * per, n_seg = max(0, min(per, c.n_chunks - c0));
  const int n_spill = c.spill_cap > 0 ? c.spill_count[q] : 0;
  bool over = n_spill > c.spill_cap;
  int total = 0;
  if (kSeg) {
    const int n = lane < n_seg ? c.seg_count[(size_t)q * c.n_chunks + c0 + lane] : 0;
    const int m = min(n, c.seg_cap);
    int incl = m;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    off[lane] = incl - m;
    total = __shfl(incl, kWave - 1, kWave);
    over = over || (c.spill_cap == 0 && __any(n > c.seg_cap));
  }
  int all = total;
  if (kSeg && W > 1) {
    if (lane == 0) {
      tot_s[w] = total;
      over_s[w] = over ? 1 : 0;
    }
    __syncthreads();
    all = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      all += tot_s[i];
      over = over || over_s[i] != 0;
    }
  }
  if (over || all + n_spill < need) {                 // the same for every wave of the query
    if (lane == 0 && w == 0) {
      fl.flags[q] = over ? kOverflowed : kTooFew;
      atomicAdd(fl.word, 1u);
    }
    return;
  }
  if (lane == 0 && w == 0) fl.flags[q] = kNotFlagged;
  __builtin_amdgcn_wave_barrier();                    // off[] written before it is read

  TopList<S> top(pend[wg]);
  constexpr int kPre = W == 1 ? 8 : 4;                // loads in flight per wave
  const uint64_t* src = c.seg + ((size_t)q * c.n_chunks + c0) * c.seg_cap;
  for (int e0 = 0; kSeg && e0 < total; e0 += kWave * kPre) {
    uint64_t cur[kPre];
#pragma unroll
    for (int j = 0; j < kPre; ++j) {
      const int e = e0 + kWave * j + lane;
      cur[j] = kPadKey;
      if (e < total) {
        int lo = 0, hi = n_seg - 1;                   // the last segment l with off[l] <= e
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (off[mid] <= e) lo = mid; else hi = mid - 1;
        }
        cur[j] = src[(size_t)lo * c.seg_cap + (e - off[lo])];
      }
    }
#pragma unroll
    for (int j = 0; j < kPre; ++j) top.take(cur[j]);
  }
  const uint64_t* more = c.spill + (size_t)q * c.spill_cap;
  for (int e0 = w * kWave; e0 < n_spill; e0 += kPre * W * kWave) {
    uint64_t cur[kPre];
#pragma unroll
    for (int j = 0; j < kPre; ++j) {
      const int e = e0 + j * W * kWave + lane;
      cur[j] = e < n_spill ? more[e] : kPadKey;
    }
#pragma unroll
    for (int j = 0; j < kPre; ++j) top.take(cur[j]);
  }
  top.flush();
  if constexpr (W > 1) {
    merge_lists<S, W>(top.lv, &lists[0][0], w, W);
    if (w != 0) return;
  }
  top.write(k, ids + (size_t)q * k, sims + (size_t)q * k);
}

// Wavefronts per query: 16 while the workgroups of 16 fit the chip at once
// (256 of them), 4 while the queries are fewer than the chip's 2,048 resident
// workgroups of 4, else 1 (1,001 queries of about 700 candidates: 1 wave
// 18.7 us, 4 waves 12.3; 100 of about 2,100: 1 wave 34.2 us, 16 waves 15.7).
int select_waves(int Q) { return Q <= 256 ? 16 : (Q <= 2048 ? 4 : 1); }

template <int S>
void launch_s(const Candidates& c, int Q, int k, int need, Flagged fl, int32_t* ids, float* sims,
              hipStream_t stream) {
  const int waves = select_waves(Q);
  if (c.n_chunks == 0)
    hipLaunchKernelGGL((select_kernel<S, 16, false>), dim3(Q), dim3(1024), 0, stream, c, Q, k, need, fl, ids, sims);
  else if (waves == 16)
    hipLaunchKernelGGL((select_kernel<S, 16, true>), dim3(Q), dim3(1024), 0, stream, c, Q, k, need, fl, ids, sims);
  else if (waves == 4)
    hipLaunchKernelGGL((select_kernel<S, 4, true>), dim3(Q), dim3(256), 0, stream, c, Q, k, need, fl, ids, sims);
  else
    hipLaunchKernelGGL((select_kernel<S, 1, true>), dim3((Q + 3) / 4), dim3(256), 0, stream, c, Q, k, need, fl, ids,
                       sims);
}

}  // namespace

hipError_t launch_select(const Candidates& c, int Q, int k, int need, Flagged fl, int32_t* ids, float* sims,
                         hipStream_t stream) {
  if (Q == 0) return hipSuccess;
  // A wave holds the counts of its share of the segments one per lane.
  if (k < 1 || k > 256 || c.n_chunks < 0 || c.n_chunks > kWave * select_waves(Q)) return hipErrorInvalidValue;
  LaunchScope scope("topk_select", stream);
  if (k <= 64) launch_s<1>(c, Q, k, need, fl, ids, sims, stream);
  else if (k <= 128) launch_s<2>(c, Q, k, need, fl, ids, sims, stream);
  else launch_s<4>(c, Q, k, need, fl, ids, sims, stream);
  return hipGetLastError();
}

}  // namespace sage
