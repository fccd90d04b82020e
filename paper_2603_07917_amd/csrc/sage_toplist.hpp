// A wavefront's running list of its S * 64 best neighbour keys, and the merge
// of several wavefronts' lists (used by the candidate selects).
#pragma once
#include "sage_device.hpp"

namespace sage {

// The list is descending over positions p = 64 s + lane (register s, lane).
// Half-cleaners sort a bitonic list.
template <int S>
__device__ __forceinline__ void list_clean(uint64_t (&lv)[S]) {
#pragma unroll
  for (int st = S / 2; st >= 1; st >>= 1)
#pragma unroll
    for (int s = 0; s < S; ++s)
      if ((s & st) == 0) {
        const uint64_t x = lv[s], y = lv[s + st];
        lv[s] = x > y ? x : y;
        lv[s + st] = x > y ? y : x;
      }
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int stride = 32; stride > 0; stride >>= 1) lv[s] = cx_lanes(lv[s], stride, true);
}
// Fold 64 keys (one per lane, any order) into the list: sorted ascending
// they are the reversed tail of a descending list, so max(A_p, B_(KL-1-p))
// touches the last register only and leaves a bitonic list.
template <int S>
__device__ __forceinline__ void list_fold(uint64_t (&lv)[S], uint64_t key) {
  const uint64_t asc = wave_sort64(key, false);
  lv[S - 1] = lv[S - 1] > asc ? lv[S - 1] : asc;
  list_clean<S>(lv);
}

// Keys that beat the list's last key are gathered in the wave's `pend` (2 x 64
// keys of LDS) and folded 64 at a time, so that of n keys about
// KL (1 + ln(n / KL)) are sorted.
template <int S>
struct TopList {
  uint64_t lv[S];
  uint64_t* buf;
  int n_buf = 0;                                      // keys waiting in buf (wave-uniform, < 64)
  __device__ __forceinline__ explicit TopList(uint64_t* pend) : buf(pend) {
#pragma unroll
    for (int s = 0; s < S; ++s) lv[s] = kPadKey;
  }
  // 64 keys, one per lane (kPadKey: none). Every lane of the wave calls it.
  __device__ __forceinline__ void take(uint64_t cur) {
    const int lane = (int)lane_id();
    const bool keep = cur > lane_value_u64(lv[S - 1], kWave - 1);
    const uint64_t mask = __ballot(keep);
    if (mask == 0) return;
    const int pos = n_buf + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    if (keep) buf[pos] = cur;
    n_buf += __popcll(mask);
    __builtin_amdgcn_wave_barrier();
    if (n_buf >= kWave) {                             // fold 64, keep the rest (< 64) at the front
      list_fold<S>(lv, buf[lane]);
      n_buf -= kWave;
      const uint64_t rest = lane < n_buf ? buf[kWave + lane] : kPadKey;
      __builtin_amdgcn_wave_barrier();
      if (lane < n_buf) buf[lane] = rest;
      __builtin_amdgcn_wave_barrier();
    }
  }
  __device__ __forceinline__ void flush() {
    const int lane = (int)lane_id();
    if (n_buf > 0) list_fold<S>(lv, lane < n_buf ? buf[lane] : kPadKey);
    n_buf = 0;
  }
  __device__ __forceinline__ void write(int k, int32_t* ids, float* sims) const {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int p = 64 * s + (int)lane_id();
      if (p < k) {
        ids[p] = lv[s] == kPadKey ? -1 : key_id(lv[s]);
        sims[p] = lv[s] == kPadKey ? -__builtin_inff() : key_sim(lv[s]);
      }
    }
  }
};

// Pairwise tree over the workgroup's W waves, of which the first `used` may
// hold keys: C_p = max(A_p, B_(KL-1-p)) is bitonic and holds the KL best of
// both. Wave 0 ends with the result. `lists`: W x KL keys of LDS. Every thread
// of the workgroup calls it.
template <int S, int W>
__device__ __forceinline__ void merge_lists(uint64_t (&lv)[S], uint64_t* lists, int w, int used) {
  constexpr int KL = 64 * S;
  const int lane = (int)lane_id();
#pragma unroll
  for (int s = 0; s < S; ++s) lists[w * KL + 64 * s + lane] = lv[s];
  __syncthreads();
  for (int h = 1; h < W && h < used; h <<= 1) {
    if ((w & (2 * h - 1)) == 0) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const uint64_t o = lists[(w + h) * KL + 64 * (S - 1 - s) + (kWave - 1 - lane)];
        lv[s] = lv[s] > o ? lv[s] : o;
      }
      list_clean<S>(lv);
#pragma unroll
      for (int s = 0; s < S; ++s) lists[w * KL + 64 * s + lane] = lv[s];
    }
    __syncthreads();
  }
}

}  // namespace sage
