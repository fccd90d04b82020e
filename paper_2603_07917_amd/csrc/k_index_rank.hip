// Gittins index scan (with the cost model fused in) and the radix-sort rank.
#include <algorithm>
#include "sage_device.hpp"
#include "sage_internal.hpp"

namespace sage {
namespace {

// ---------------------------------------------------------------------------
// Index scan. G lanes per request row (64 / G rows per wavefront); lane l of
// a row owns the C consecutive bins [l*C, l*C + C), C G >= B.
//   F_b = sum_{j<=b} p_j, S_b = sum_{j<=b} p_j x_j, T_b = sum_{j>b} p_j,
//   G = min over b with F_b > 0 of (S_b + T_b x_b) / F_b.
// Candidates are compared by cross-multiplication (N_b F* < N* F_b), so a lane
// costs one fp64 division. All sums are fp64.
//
// Bound by the issue of fp64 instructions: about 17 per bin, and per wave
// about 110 for the scans, the division and the minimum over lanes. Rows of
// up to 512 bins therefore take 16 or 32 lanes and share that part (against 64
// lanes a row, same box: 20,011 x 256 10.8 -> 8.1 us, 65,536 x 512 38.9 ->
// 33.5 us; 65,536 x 1,024 69.0 -> 65.5 us from scalar prompt lengths, late
// stores and the fp32 minimum; refresh table 32,768 x 256 x 41 429 -> 118 us).
// ---------------------------------------------------------------------------
template <int C, bool kFull>
__device__ __forceinline__ void load_row(const float* __restrict__ mass, size_t row, int b0, int B,
                                         float (&p)[C]) {
  if (kFull && C % 4 == 0) {
#pragma unroll
    for (int j = 0; j < C; j += 4) {
      const float4 v = *reinterpret_cast<const float4*>(mass + row + b0 + j);
      p[j] = v.x; p[j + 1] = v.y; p[j + 2] = v.z; p[j + 3] = v.w;
    }
  } else if (!kFull && C % 4 == 0 && B % 4 == 0) {   // rows 16-byte aligned, no quad crosses the row's end
#pragma unroll
    for (int j = 0; j < C; j += 4) {
      float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (b0 + j < B) v = *reinterpret_cast<const float4*>(mass + row + b0 + j);
      p[j] = v.x; p[j + 1] = v.y; p[j + 2] = v.z; p[j + 3] = v.w;
    }
  } else if (C % 4 == 0) {                           // four at a time from 4-byte aligned addresses
#pragma unroll
    for (int j = 0; j < C; j += 4) {
      if (kFull || b0 + j + 3 < B) {
        float v[4];
        __builtin_memcpy(v, mass + row + b0 + j, sizeof v);
        p[j] = v[0]; p[j + 1] = v[1]; p[j + 2] = v[2]; p[j + 3] = v[3];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[j + i] = b0 + j + i < B ? mass[row + b0 + j + i] : 0.0f;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < C; ++j) p[j] = (kFull || b0 + j < B) ? mass[row + b0 + j] : 0.0f;
  }
}

// kFull: B == C G, so every lane owns C real bins (no guards, vector loads).
// kMode: kGivenCost takes the support from the cost matrix; kFused computes
// it from the prompt length and the representatives (kept in LDS);
// kAttained also refreshes running requests: with o = bucket *
// floor(generated / bucket) tokens served, a = o^2 / 2 + I o, the bins with
// x <= a are ruled out and the rest are shifted down by a, so the result is
// the index of the remaining cost. kVariant takes the cost model, the kind
// of index (Gittins or mean) and a uniform-mixing weight at run time.
// kTable: kAttained for every row at each level o = lv * bucket (lv < levels),
// one row per wave and 64 / G levels at a time. kTableRows: the same with 64 / G
// rows per wave and one level at a time, for tables of few levels, which would
// leave some of a row's lane groups without one (and have no long run of levels
// past all mass to skip). Both give kAttained's bits.
enum IndexMode { kGivenCost = 0, kFused = 1, kAttained = 2, kVariant = 3, kTable = 4, kTableRows = 5 };
constexpr int kTableRowsMax = 5;     // levels
// Workgroups per CU the register budget is tuned for (4 waves each).
// The table keeps its support in registers: 2 of them and no spills at C = 16.
template <int C, int kMode> struct IndexOcc {
  static constexpr int value = C <= 8 ? 4 : (C == 16 ? (kMode >= 4 ? 2 : 3) : 1);
};

constexpr int kNoBin = 0x7fffffff;   // a lane without a candidate bin

template <int C, int G, bool kFull, int kMode, bool kArg>
__global__ void __launch_bounds__(256, (IndexOcc<C, kMode>::value)) index_kernel(const float* __restrict__ mass,
                                                    const float* __restrict__ cost,
                                                    const int32_t* __restrict__ prompt_len,
                                                    const double* __restrict__ repr,
                                                    const int32_t* __restrict__ generated, int bucket,
                                                    int Q, int B, float* __restrict__ index,
                                                    int32_t* __restrict__ argmin, IndexVariant var) {
  constexpr bool kFused = kMode != kGivenCost;
  constexpr bool kAtt = kMode == kAttained || kMode == kTable || kMode == kTableRows;
  constexpr int kR = kWave / G;                    // rows, or levels of a row, at a time
  constexpr int kRows = kMode == kTable ? 1 : kR;  // rows per wave and turn
  // Representatives (fused cost only): lane l's C of them at l * kPitch. Without
  // the pad every lane of a read would start on one or a few of the 64 banks
  // (C = 16: two of them).
  constexpr int kPitch = C >= 4 ? C + 2 : C;
  extern __shared__ __align__(16) double repr_s[];
  const int lane = (int)lane_id();
  const int group = lane / G, l = lane % G;
  // Uniform over the wave.
  const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave));
  const int q_step = (int)(gridDim.x * (blockDim.x / kWave)) * kRows;
  const int b0 = l * C;
  const double* repr_l = repr_s + l * kPitch;      // element j: bin b0 + j (valid below B)
  const int q_first = wave * kRows;
  // This lane's row of a turn (rows past the last one repeat it, unstored).
  auto row_of = [&](int base) { return kRows == 1 ? base : min(base + group, Q - 1); };

  float p[C], p_next[C];
  int I_next = 0;
  // A given cost row that does not fill its lanes is loaded as the masses are
  // (C <= 32): read one by one where used, the 16 consecutive costs of each of 64
  // lanes took 65,536 rows of 200 bins 74 us, so 18, and 1,500 bins 802, so 168;
  // full rows are as fast so (the compiler joins the reads).
  constexpr bool kKeepCost = kMode == kGivenCost && C <= 32 && !kFull;
  float x_cost[kKeepCost ? C : 1], x_next[kKeepCost ? C : 1];
  // Next row's prompt length before its masses: loads return in order.
  auto load_next = [&](int base) {
    const int q = row_of(base);
    if (kFused) I_next = prompt_len[q];
    load_row<C, kFull>(mass, (size_t)q * (size_t)B, b0, B, p_next);
    if constexpr (kKeepCost) load_row<C, kFull>(cost, (size_t)q * (size_t)B, b0, B, x_next);
  };
  if (q_first < Q) load_next(q_first);             // in flight while LDS is set up
  if (kFused) {
    for (int b = threadIdx.x; b < B; b += blockDim.x) repr_s[b / C * kPitch + b % C] = repr[b];
    __syncthreads();
  }

  // A row's result (its last lane's) is stored when the next row's loads are
  // about to go out: a wait for loads also waits for the stores issued before
  // it, and one issued just before the wait would cost its whole round trip.
  float res = 0.0f;
  int res_arg = -1, res_base = -1;
  auto store_result = [&]() {
    if (kMode != kTable && kMode != kTableRows && res_base >= 0 && l == G - 1 && res_base + group < Q) {
      index[res_base + group] = res;
      if (kArg) argmin[res_base + group] = res_arg;
    }
  };
  // Levels [lv_first, n_lv) of the table (blockIdx.y: their share).
  const int lv_first = kMode == kTable ? (int)blockIdx.y * var.level_share : 0;
  const int n_lv = kMode == kTable ? lv_first + min(var.level_share, var.levels - lv_first)
                                   : (kMode == kTableRows ? var.levels : 1);
  constexpr int kStep = kMode == kTable ? kR : 1;
  for (int base = q_first; base < Q; base += q_step) {
    const int q = row_of(base);
    const size_t row = (size_t)q * (size_t)B;
#pragma unroll
    for (int j = 0; j < C; ++j) p[j] = p_next[j];
    if constexpr (kKeepCost) {
#pragma unroll
      for (int j = 0; j < C; ++j) x_cost[j] = x_next[j];
    }
    const double I = (double)I_next;
    store_result();
    res_base = base;
    if (base + q_step < Q) load_next(base + q_step);
    // Refresh table: the support stays in registers across the levels (C <= 16, and
    // C = 32 with guards: 5,000 rows x 1,500 bins x 41 levels 817 -> 352 us; full
    // rows gain more from two waves per SIMD), and lane t keeps the result of level
    // t (mod 64), written 64 at a time.
    constexpr bool kKeepX = (kMode == kTable || kMode == kTableRows) && (C <= 16 || (C == 32 && !kFull));
    double x_row[kKeepX ? C : 1];
    if (kKeepX) {
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const double r = (kFull || b0 + j < B) ? repr_l[j] : 0.0;
        x_row[j] = r * fma(0.5, r, I);
      }
    }
    float lane_res = 0.0f;
   // Counted so that levels up to 2^31 - 1 do not run over.
   for (int step = 0; step <= (n_lv - lv_first - 1) / kStep; ++step) {
    const int lv = lv_first + step * kStep;
    double a = 0.0;                                 // service already received
    if (kAtt) {
      const double o = kMode == kTable       ? ((double)lv + (double)group) * (double)bucket
                       : kMode == kTableRows ? (double)lv * (double)bucket
                                             : (double)((max(generated[q], 0) / bucket) * bucket);
      a = o * fma(0.5, o, I);
    }

    // Support x_j = r (I + r / 2) (or the given cost); recomputed where used,
    // which keeps the register count (and so the occupancy) down.
    auto support = [&](int j) -> double {
      if (kKeepX) return x_row[kKeepX ? j : 0];
      const int b = b0 + j;
      const bool in = kFull || b < B;
      if (kMode == kVariant) {
        const double r = in ? repr_l[j] : 0.0;
        if (var.cost_model == 1) return r;                       // output length
        if (var.cost_model == 2) return fma(2.0, r, I);          // input + 2 output
        return r * fma(0.5, r, I);
      }
      if (kFused) {
        const double r = in ? repr_l[j] : 0.0;
        return r * fma(0.5, r, I);
      }
      if (kKeepCost) return (double)x_cost[kKeepCost ? j : 0];
      return in ? (double)cost[row + b] : 0.0;
    };
    if (kMode == kVariant && var.noise > 0.0f) {     // p' = (1 - w) p / sum(p) + w / B
      double raw = 0.0;
#pragma unroll
      for (int j = 0; j < C; ++j) raw += (double)p[j];
      const double tot = group_total_f64<G>(group_incl_scan_f64<G>(raw));
      if (tot > 0.0) {
        const double keep = (1.0 - (double)var.noise) / tot, spread = (double)var.noise / (double)B;
#pragma unroll
        for (int j = 0; j < C; ++j)
          if (kFull || b0 + j < B) p[j] = (float)fma(keep, (double)p[j], spread);
      }
    }
    // The mass of bin j; with attained service, the outcomes already passed
    // (x <= a) are ruled out (p itself is kept for the next level).
    auto pm = [&](int j) -> double {
      if (kAtt && !(support(j) > a)) return 0.0;
      return (double)p[j];
    };
    double lane_f = 0.0, lane_s = 0.0;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      lane_f += pm(j);
      lane_s = fma(pm(j), support(j) - a, lane_s);
    }
    // Prefix sums over the row's lanes (DPP); the mass above this lane is the
    // row total minus the inclusive prefix (fp64, so its rounding is ~1e-16 of
    // the total).
    const double f_incl = group_incl_scan_f64<G>(lane_f);
    const double f_base = group_shift_up_f64<G>(f_incl);
    const double s_base = group_shift_up_f64<G>(group_incl_scan_f64<G>(lane_s));
    const double f_total = group_total_f64<G>(f_incl);
    // No mass above a: +inf here and at every later level (a grows with the
    // level, so what it rules out stays ruled out). A row of 64 predicted
    // lengths passes its longest one after about 16 of 41 levels of 200.
    if (kMode == kTable && !__any(f_total != 0.0) && I >= 0.0) {
      for (uint32_t t = (uint32_t)((lv & ~(kWave - 1)) + lane); t < (uint32_t)n_lv; t += kWave)
        if (t >= (uint32_t)lv_first)
          index[(size_t)t * (size_t)Q + (size_t)q] = t < (uint32_t)lv ? lane_res : __builtin_inff();
      break;
    }
    if (kMode == kTableRows && __all(f_total == 0.0 && I >= 0.0)) {
      for (int t = lv + l; t < n_lv; t += G)
        if (base + group < Q) index[(size_t)t * (size_t)Q + (size_t)q] = __builtin_inff();
      break;
    }
    if (kMode == kVariant && var.kind == 1) {        // the mean: sum p x / sum p
      const double s_incl = s_base + lane_s;
      res = f_total > 0.0 ? (float)(s_incl / f_total) : __builtin_inff();   // the last lane's
      res_arg = -1;
      continue;
    }

    // Branch-free running minimum of n / f by cross-multiplication; the
    // start values (n, f) = (1, 0) lose to the first bin with f > 0 (f never
    // decreases, so no bin with f = 0 can win later), and a later bin must be
    // strictly smaller to win (ties keep the lower bin).
    double best_n = 1.0, best_f = 0.0;
    int best_b = kNoBin;
    double f_run = f_base, s_run = s_base, t_run = f_total - f_base;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const double pj = pm(j);
      const double xj = support(j) - a;
      f_run += pj;
      s_run = fma(pj, xj, s_run);
      t_run -= pj;                                  // mass strictly above bin j
      const double n = fma(t_run, xj, s_run);
      const bool take = (kFull || b0 + j < B) && n * best_f < best_n * f_run;
      best_n = take ? n : best_n;
      best_f = take ? f_run : best_f;
      if (kArg) best_b = take ? b0 + j : best_b;
    }
    // One division per lane, then the minimum of the ratios over the row's
    // lanes, complete in its last lane. With the argmin (ties keep the smaller
    // bin) in fp64: butterflies within rows of 16 (quads, half rows, rows),
    // then rows 0+1 -> 1, 2+3 -> 3 (G >= 32) and 1 -> 3 (G = 64). Lanes without
    // a candidate carry +inf and lose every tie.
    double r = best_f > 0.0 ? best_n / best_f : __builtin_inf();
    if (kArg) {
      auto combine = [&](double orr, int ob) {
        const bool take = orr < r || (orr == r && ob < best_b);
        r = take ? orr : r;
        best_b = take ? ob : best_b;
      };
#define SAGE_ARGMIN_STEP(CTRL, ROWS) \
      combine(dpp_f64<CTRL, ROWS>(r, r), (int)dpp_u32<CTRL, ROWS>((uint32_t)best_b, (uint32_t)best_b))
      SAGE_ARGMIN_STEP(kDppQuadXor1, 0xf);
      SAGE_ARGMIN_STEP(kDppQuadXor2, 0xf);
      SAGE_ARGMIN_STEP(kDppRowHalfMirror, 0xf);
      SAGE_ARGMIN_STEP(kDppRowMirror, 0xf);
      if (G >= 32) SAGE_ARGMIN_STEP(kDppRowBcast15, 0xa);
      if (G == 64) SAGE_ARGMIN_STEP(kDppRowBcast31, 0xc);
#undef SAGE_ARGMIN_STEP
      const bool found = r < __builtin_inf();
      res = found ? (float)r : __builtin_inff();
      res_arg = found ? best_b : -1;
    } else {
      // Without it, of the lanes' fp32 values (the rounding is monotone, so it
      // commutes with the minimum) as monotone bits: one DPP minimum per step
      // where fp64 takes six instructions.
      res = f32_from_order_bits(group_min_u32<G>(f32_order_bits((float)r)));
    }
    if (kMode == kTableRows && l == G - 1 && base + group < Q) index[(size_t)lv * (size_t)Q + (size_t)q] = res;
    if (kMode == kTable) {
      const int t0 = lv & (kWave - 1);                // lv is a multiple of kR, which divides 64
#pragma unroll
      for (int g = 0; g < kR; ++g) {
        const float v = __uint_as_float(
            (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(res), g * G + G - 1));
        if (lane == t0 + g) lane_res = v;
      }
      if (t0 + kR == kWave || n_lv - lv <= kR) {
        const int t = (lv & ~(kWave - 1)) + lane;
        if (t >= lv_first && t - lv < kR && t < n_lv) index[(size_t)t * (size_t)Q + (size_t)q] = lane_res;
      }
    }
   }
  }
  store_result();
}

template <int C, int G, bool kFull, int kMode>
hipError_t launch_index_v(const float* mass, const float* cost, const int32_t* prompt_len,
                          const double* repr, const int32_t* generated, int bucket, int Q, int B,
                          float* index, int32_t* argmin, hipStream_t stream, IndexVariant var) {
  const int waves_per_block = 4;
  // One turn per wave up to a number of workgroups, then several, the next row
  // loading behind the one being scanned: a new workgroup first stages the
  // representatives (65,536 rows x 1,024 bins: 2,048 workgroups 65.6 us, 4,096
  // 67.1, 16,384 81; mean of 65,536 x 512: 2,048 27.6, 4,096 29.0; table of 32,768
  // rows x 41 levels: 1,024 workgroups 126 us, 2,048 118, 4,096 125, 8,192 138).
  // Where a wave takes much of the register file, one round of them (but for the
  // table, whose rows take unequal time): one a CU at C = 64 and two at C = 32
  // (16,384 x 4,096: 2,048 workgroups 101 us, 256 59; with attained service 246
  // and 169; 16,384 x 2,048 52 and 41).
  const long most = kMode >= kTable ? 2048 : C >= 64 ? 256 : C == 32 ? 512
                    : C * G == 512 || (C * G >= 1024 && kMode != kGivenCost) ? 2048 : 4096;
  const int rows = waves_per_block * (kMode == kTable ? 1 : kWave / G);
  const long blocks = std::min<long>(((long)Q + rows - 1) / rows, most);
  // Table of few rows: their levels in shares (multiples of 64 / G), while the
  // waves are fewer than four a CU. One row of 2,048 bins and 41 levels took
  // one wave 79 us, shared 7.5.
  unsigned shares = 1;
  if (kMode == kTable) {
    const long want = std::max(1L, 256 / blocks), steps = ((long)var.levels + kWave / G - 1) / (kWave / G);
    const long share = (steps + std::min(want, steps) - 1) / std::min(want, steps) * (kWave / G);
    var.level_share = (int)std::min<long>(share, var.levels);
    shares = (unsigned)((var.levels - 1) / var.level_share + 1);
  }
  // Representatives, a pitch of C + 2 per lane that has any (C as it is for C < 4).
  const size_t lds = kMode != kGivenCost ? (size_t)((B + C - 1) / C) * (C >= 4 ? C + 2 : C) * sizeof(double) : 0;
  const dim3 grid((unsigned)blocks, shares);
  if (argmin && kMode < kTable)                      // the tables have none
    hipLaunchKernelGGL((index_kernel<C, G, kFull, kMode, kMode < kTable>), grid, dim3(64 * waves_per_block), lds,
                       stream, mass, cost, prompt_len, repr, generated, bucket, Q, B, index, argmin, var);
  else
    hipLaunchKernelGGL((index_kernel<C, G, kFull, kMode, false>), grid, dim3(64 * waves_per_block), lds, stream, mass,
                       cost, prompt_len, repr, generated, bucket, Q, B, index, argmin, var);
  return hipGetLastError();
}

template <int C, int G>
hipError_t launch_index_c(const float* mass, const float* cost, const int32_t* prompt_len,
                          const double* repr, const int32_t* generated, int bucket, int Q, int B,
                          float* index, int32_t* argmin, hipStream_t stream, const IndexVariant* variant) {
  const bool full = B == C * G;
  const int mode = (variant && variant->levels > 0) ? kTable
                   : variant ? kVariant : (generated ? kAttained : (cost ? kGivenCost : kFused));
  const IndexVariant var = variant ? *variant : IndexVariant();
#define SAGE_INDEX_LAUNCH(FULL, MODE)                                                               \
  return launch_index_v<C, G, FULL, MODE>(mass, cost, prompt_len, repr, generated, bucket, Q, B, index, \
                                       argmin, stream, var)
  if (mode == kVariant) {
    if (full) SAGE_INDEX_LAUNCH(true, kVariant);
    SAGE_INDEX_LAUNCH(false, kVariant);
  }
  if constexpr (G < kWave) {
    // 65,536 rows x 256 bins: one level 63 -> 19 us (64 lanes a row: 28), two
    // 63 -> 28 (47); 512 bins: three 105 -> 73 (85), five 146 -> 113 (136).
    if (mode == kTable && var.levels <= kTableRowsMax) {
      if (full) SAGE_INDEX_LAUNCH(true, kTableRows);
      SAGE_INDEX_LAUNCH(false, kTableRows);
    }
  }
  if (mode == kTable) {
    if (full) SAGE_INDEX_LAUNCH(true, kTable);
    SAGE_INDEX_LAUNCH(false, kTable);
  }
  if (full) {
    if (mode == kAttained) SAGE_INDEX_LAUNCH(true, kAttained);
    if (mode == kFused) SAGE_INDEX_LAUNCH(true, kFused);
    SAGE_INDEX_LAUNCH(true, kGivenCost);
  }
  if (mode == kAttained) SAGE_INDEX_LAUNCH(false, kAttained);
  if (mode == kFused) SAGE_INDEX_LAUNCH(false, kFused);
  SAGE_INDEX_LAUNCH(false, kGivenCost);
#undef SAGE_INDEX_LAUNCH
}

// ---------------------------------------------------------------------------
// Rank: stable least-significant-digit radix sort of the index keys (fp32
// bits made monotone, -0 folded onto +0), 8-bit digits, 4 passes. Each pass:
// per-tile digit counts, one exclusive scan over (digit, tile), then a stable
// scatter where each wave ranks equal digits of its own quarter of the tile
// with ballots (three barriers a tile; with three for every 256 requests and
// the scatter's own sum of the counts, 1.34 M keys took 14.4 us a scatter, now
// 11.7, and 131,073 keys 88 us in all, now 54).
// ---------------------------------------------------------------------------
constexpr int kRankThreads = 256;
constexpr int kRankItems = 8;
constexpr int kRankTile = kRankThreads * kRankItems;

__device__ __forceinline__ uint32_t index_key(float g) {
  uint32_t u = __float_as_uint(g);
  if (u == 0x80000000u) u = 0u;      // -0 sorts with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__global__ void __launch_bounds__(kRankThreads) rank_hist_kernel(const float* __restrict__ g_in,
                                                                 const uint32_t* __restrict__ k_in,
                                                                 int Q, int shift, int n_tiles,
                                                                 uint32_t* __restrict__ hist) {
  __shared__ uint32_t cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * kRankTile;
#pragma unroll
  for (int it = 0; it < kRankItems; ++it) {
    const int i = base + it * kRankThreads + threadIdx.x;
    const bool in = i < Q;
    const uint32_t digit = in ? ((k_in ? k_in[i] : index_key(g_in[i])) >> shift) & 255u : 256u;
    // A wave of one digit (runs of equal keys: exhausted requests at +inf)
    // counts it once; 64 atomics on one word would queue up.
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)digit);
    if (__all(digit == d0)) {
      if (d0 < 256u && lane_id() == 0) atomicAdd(&cnt[d0], (uint32_t)kWave);
    } else if (in) {
      atomicAdd(&cnt[digit], 1u);
    }
  }
  __syncthreads();
  hist[threadIdx.x * n_tiles + blockIdx.x] = cnt[threadIdx.x];
}

// Per-digit exclusive scan over the tiles: workgroup d scans hist[d][0..n_tiles)
// in place (contiguous, 256 counts per turn) and leaves the digit's total in
// total[d]. The scatter adds the exclusive scan of the 256 totals.
__global__ void __launch_bounds__(256) rank_scan_kernel(uint32_t* __restrict__ hist, int n_tiles,
                                                        uint32_t* __restrict__ total) {
  __shared__ uint32_t wsum[4];
  const int t = threadIdx.x;
  const int lane = (int)lane_id();
  const int w = t / kWave;
  uint32_t* row = hist + (size_t)blockIdx.x * n_tiles;
  uint32_t carry = 0;
  for (int base = 0; base < n_tiles; base += 256) {
    const int i = base + t;
    const uint32_t v = i < n_tiles ? row[i] : 0u;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)incl, o, kWave);
      if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t before = carry;
    for (int ww = 0; ww < w; ++ww) before += wsum[ww];
    if (i < n_tiles) row[i] = before + incl - v;
    carry += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
  if (t == 0) total[blockIdx.x] = carry;
}

__global__ void __launch_bounds__(kRankThreads) rank_scatter_kernel(
    const float* __restrict__ g_in, const uint32_t* __restrict__ k_in,
    const uint32_t* __restrict__ v_in, int Q, int shift, int n_tiles,
    const uint32_t* __restrict__ offsets, const uint32_t* __restrict__ digit_total,
    uint32_t* __restrict__ k_out, uint32_t* __restrict__ v_out) {
  constexpr int kWaves = kRankThreads / kWave;
  __shared__ uint32_t base_off[256];
  __shared__ uint32_t wtot[kWaves];
  __shared__ uint32_t cnt[kWaves][256];
  const int t = threadIdx.x;
  const int lane = (int)lane_id();
  const int w = __builtin_amdgcn_readfirstlane(t / kWave);
  // Wave w owns the w-th quarter of the tile (kRankItems turns of 64 requests,
  // in order): it ranks its requests among its own by digit with no barrier,
  // and the waves' counts are combined once.
  const int first = blockIdx.x * kRankTile + w * (kRankItems * kWave) + lane;
  uint32_t key[kRankItems], val[kRankItems];
#pragma unroll
  for (int it = 0; it < kRankItems; ++it) {
    const int i = first + it * kWave;
    const bool valid = i < Q;
    key[it] = valid ? (k_in ? k_in[i] : index_key(g_in[i])) : 0u;
    val[it] = valid ? (v_in ? v_in[i] : (uint32_t)i) : 0u;
  }
  // Exclusive scan of the 256 digit totals (one per thread), plus this tile's
  // offset within the digit.
  {
    const uint32_t v = digit_total[t], tile_off = offsets[t * n_tiles + blockIdx.x];
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)incl, o, kWave);
      if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) wtot[w] = incl;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) cnt[i][t] = 0;
    __syncthreads();
    uint32_t before = 0;
    for (int ww = 0; ww < w; ++ww) before += wtot[ww];
    base_off[t] = before + incl - v + tile_off;
  }
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint32_t rank[kRankItems];                       // among the wave's requests of the same digit
#pragma unroll
  for (int it = 0; it < kRankItems; ++it) {
    const bool valid = first + it * kWave < Q;
    const uint32_t digit = (key[it] >> shift) & 255u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool on = (digit >> bit) & 1u;
      const uint64_t m = __ballot(on);
      peers &= on ? m : ~m;
    }
    const uint32_t seen = cnt[w][digit];           // LDS operations of a wave complete in order
    rank[it] = seen + (uint32_t)__popcll(peers & lt_mask);
    __builtin_amdgcn_wave_barrier();
    if (valid && (peers & lt_mask) == 0) cnt[w][digit] = seen + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  {
    uint32_t run = base_off[t];                    // counts -> first positions, wave by wave
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      const uint32_t c = cnt[ww][t];
      cnt[ww][t] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kRankItems; ++it) {
    if (first + it * kWave >= Q) continue;
    const uint32_t pos = cnt[w][(key[it] >> shift) & 255u] + rank[it];
    if (k_out) k_out[pos] = key[it];
    v_out[pos] = val[it];
  }
}

// Rank of a small queue (Q <= kRankSmallMax) by counting: the position of
// request i in the stable ascending order is
//   rank(i) = #{j : key_j < key_i} + #{j < i : key_j == key_i},
// the same permutation the radix sort gives. Workgroup b owns TI requests
// i0 = TI b ... and counts over all Q keys, held in LDS: its 16 waves take
// 64-key chunks in turn, and within a wave S = 64 / TI lane groups take
// TI-key sub-blocks of each chunk (lane l: request i0 + l % TI, sub-block
// l / TI). A chunk wholly below i0 counts key_j <= key_i, one wholly past
// the workgroup's requests counts key_j < key_i, and only the chunk holding
// them takes the exact rule. Q^2 compares, one compare and one add each:
// at these sizes a few microseconds spread over the whole chip, where the
// four-pass radix sort in one workgroup ran serially.
constexpr int kRankSmallMax = 8192;
constexpr int kRankCountThreads = 1024;
constexpr int kRankCountWaves = kRankCountThreads / kWave;

template <int TI>
__global__ void __launch_bounds__(kRankCountThreads) rank_count_kernel(const float* __restrict__ g_in, int Q,
                                                                       int32_t* __restrict__ order) {
  constexpr int S = kWave / TI;
  __shared__ __align__(16) uint32_t keys[kRankSmallMax];
  __shared__ uint32_t part[kRankCountWaves][TI];
  const int tid = threadIdx.x;
  const int lane = (int)lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);     // wave-uniform: scalar loop control
  const int n_chunks = (Q + kWave - 1) / kWave;
  {
    // All loads in flight at once, then the LDS writes; padding never counts.
    constexpr int kItems = kRankSmallMax / kRankCountThreads;
    float g[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const int e = r * kRankCountThreads + tid;
      g[r] = e < Q ? g_in[e] : 0.0f;
    }
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const int e = r * kRankCountThreads + tid;
      if (e < n_chunks * kWave) keys[e] = e < Q ? index_key(g[r]) : 0xFFFFFFFFu;
    }
  }
  __syncthreads();
  const int i0 = blockIdx.x * TI;
  const int il = lane % TI, sub = lane / TI;
  const int i = i0 + il;
  const uint32_t ki = keys[min(i, Q - 1)];
  const int c_lo = i0 / kWave;                                // chunk holding the requests
  uint32_t cnt = 0;
  for (int c = w; c < n_chunks; c += kRankCountWaves) {
    const int j0 = c * kWave + sub * TI;
    const uint4* kp = reinterpret_cast<const uint4*>(&keys[j0]);
    if (c < c_lo) {
#pragma unroll
      for (int m = 0; m < TI / 4; ++m) {
        const uint4 k4 = kp[m];
        cnt += (k4.x <= ki) + (k4.y <= ki) + (k4.z <= ki) + (k4.w <= ki);
      }
    } else if (c > c_lo) {
#pragma unroll
      for (int m = 0; m < TI / 4; ++m) {
        const uint4 k4 = kp[m];
        cnt += (k4.x < ki) + (k4.y < ki) + (k4.z < ki) + (k4.w < ki);
      }
    } else {
#pragma unroll
      for (int m = 0; m < TI; ++m) {
        const uint32_t kj = keys[j0 + m];
        cnt += (kj < ki || (kj == ki && j0 + m < i)) ? 1u : 0u;
      }
    }
  }
#pragma unroll
  for (int o = TI; o < kWave; o <<= 1) cnt += __shfl_xor(cnt, o, kWave);
  if (sub == 0) part[w][il] = cnt;
  __syncthreads();
  if (tid < TI && i < Q) {
    uint32_t r = 0;
#pragma unroll
    for (int ww = 0; ww < kRankCountWaves; ++ww) r += part[ww][tid];
    order[r] = i;
  }
}

// ---------------------------------------------------------------------------
// Rank of a medium queue (kRankSmallMax < Q <= kRankMergeMax): sorted tiles,
// then every request's position by binary searches in all of them. Two
// launches, where the radix sort takes eight (four digits, each a count and a
// scatter on a few workgroups).
//
// rank_tile_kernel: a workgroup sorts a tile of T consecutive requests by
// (key, id): each wave sorts 64 (bitonic, across lanes), and a request's place
// in the tile is its place in its wave plus, for every other wave, the number
// of its keys before it: key <= its own in an earlier wave, < in a later one
// (ids rise with the wave). Keys and ids go out in sorted order, the last tile
// padded with the largest key.
//
// rank_merge_kernel: the same rule over tiles gives the final position. A
// workgroup takes E requests of one tile; 1024 / E threads share a request,
// each searching its part of the tiles, whose keys pass through LDS in groups
// of kGroupTiles. Neighbouring lanes hold neighbouring keys, so their searches
// read mostly the same words. The work grows as Q^2 / T: 20,011 requests 56.8
// (radix) -> 11.6 us, 65,536 72.8 -> 21.8, 131,072 88.2 -> 44.9, but 160,000
// 67.6 -> 89.7. Below kRankSmallMax one launch of counting is as fast (8,192:
// 8.9 against 9.1 us; 16,384: 24.1 against 10.2).
// ---------------------------------------------------------------------------
constexpr int kRankMergeMax = 131072;
constexpr uint32_t kRankPad = 0xFFFFFFFFu;          // above every key but that of the NaN 0x7fffffff, which is it

// Number of the n (a power of two) ascending keys of `a` below k (or, with
// `or_equal`, at most k).
__device__ __forceinline__ int count_before(const uint32_t* a, int n, uint32_t k, bool or_equal) {
  // key <= k is key < k + 1 except at k = 2^32 - 1, where all are at most k.
  const uint32_t lim = or_equal ? k + 1u : k;
  if (or_equal && lim == 0u) return n;
  int pos = 0;
  for (int step = n >> 1; step > 0; step >>= 1) pos += a[pos + step - 1] < lim ? step : 0;
  return pos + (a[pos] < lim ? 1 : 0);
}

template <int T>
__global__ void __launch_bounds__(T) rank_tile_kernel(const float* __restrict__ g_in, int Q,
                                                      uint32_t* __restrict__ keys_out, int32_t* __restrict__ ids_out) {
  constexpr int kWaves = T / kWave;
  __shared__ uint32_t keys[T];
  const int lane = (int)lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int base = blockIdx.x * T;
  const int i = base + (int)threadIdx.x;
  // Sorted ascending by (key, place): the pads keep distinct places.
  const uint64_t mine = wave_sort64(((uint64_t)(i < Q ? index_key(g_in[i]) : kRankPad) << 32) | threadIdx.x, false);
  const uint32_t key = (uint32_t)(mine >> 32);
  keys[threadIdx.x] = key;
  __syncthreads();
  int pos = lane;
#pragma unroll
  for (int o = 0; o < kWaves; ++o)
    if (o != w) pos += count_before(keys + o * kWave, kWave, key, o < w);
  keys_out[base + pos] = key;
  ids_out[base + pos] = base + (int)(uint32_t)mine;
}

template <int T, int E>
__global__ void __launch_bounds__(1024) rank_merge_kernel(const uint32_t* __restrict__ keys_in,
                                                          const int32_t* __restrict__ ids_in, int Q, int n_tiles,
                                                          int32_t* __restrict__ order) {
  constexpr int kGroupTiles = 32768 / T;            // 128 KiB of keys in LDS at a time
  constexpr int kShare = 1024 / E;                  // threads per request
  constexpr int kIlp = 4;                           // searches of a thread in flight
  __shared__ __align__(16) uint32_t keys[kGroupTiles * T];
  __shared__ int part[kShare][E];
  const int e = (int)threadIdx.x % E, s = (int)threadIdx.x / E;
  const int at = blockIdx.x * E + e;                // place among the sorted tiles
  const int own = blockIdx.x * E / T;               // E divides T
  const uint32_t k = keys_in[at];
  int cnt = s == 0 ? at - own * T : 0;              // place in its own tile
  for (int t0 = 0; t0 < n_tiles; t0 += kGroupTiles) {
    const int n = min(kGroupTiles, n_tiles - t0);
    __syncthreads();                                // the previous group's searches are done
    const uint4* src = reinterpret_cast<const uint4*>(keys_in + (size_t)t0 * T);
    for (int i = threadIdx.x; i < n * T / 4; i += 1024) reinterpret_cast<uint4*>(keys)[i] = src[i];
    __syncthreads();
    for (int t = s; t < n; t += kShare * kIlp) {
      // kIlp tiles t, t + kShare, ...: the same search steps on each. A tile
      // past the group searches the last one, uncounted.
      const uint32_t* a[kIlp];
      uint32_t lim[kIlp];
      int pos[kIlp];
#pragma unroll
      for (int u = 0; u < kIlp; ++u) {
        const int tt = min(t + u * kShare, n - 1);
        a[u] = keys + tt * T;
        lim[u] = t0 + tt < own ? k + 1u : k;
        pos[u] = 0;
      }
#pragma unroll
      for (int step = T / 2; step > 0; step >>= 1)
#pragma unroll
        for (int u = 0; u < kIlp; ++u) pos[u] += a[u][pos[u] + step - 1] < lim[u] ? step : 0;
#pragma unroll
      for (int u = 0; u < kIlp; ++u) {
        pos[u] += a[u][pos[u]] < lim[u] ? 1 : 0;
        const int tt = t + u * kShare;
        if (tt < n && t0 + tt != own) cnt += pos[u];
      }
    }
  }
  // Of the tiles before, every key comes before one of kRankPad's bits (one NaN's);
  // k + 1 wraps to 0 there, so that the searches above counted none of them.
  if (s == 0 && k == kRankPad) cnt += own * T;
  part[s][e] = cnt;
  __syncthreads();
  if (s != 0) return;
  int rank = 0;
#pragma unroll
  for (int i = 0; i < kShare; ++i) rank += part[i][e];
  const int id = ids_in[at];
  if (id < Q) order[rank] = id;                     // not a pad
}

template <int T, int E>
void launch_rank_merge(const float* index, int Q, int32_t* order, void* ws, hipStream_t stream) {
  const int n_tiles = (Q + T - 1) / T;
  uint32_t* keys = static_cast<uint32_t*>(ws);
  int32_t* ids = reinterpret_cast<int32_t*>(keys + (size_t)n_tiles * T);
  {
    LaunchScope scope("rank_tiles", stream);
    hipLaunchKernelGGL(rank_tile_kernel<T>, dim3(n_tiles), dim3(T), 0, stream, index, Q, keys, ids);
  }
  LaunchScope scope("rank_merge", stream);
  hipLaunchKernelGGL((rank_merge_kernel<T, E>), dim3(n_tiles * (T / E)), dim3(1024), 0, stream, keys, ids, Q, n_tiles,
                     order);
}

}  // namespace

size_t rank_workspace_bytes(int Q) {
  if (Q <= 0) return 0;
  const size_t tiles = ((size_t)Q + kRankTile - 1) / kRankTile;
  return 4 * (size_t)Q * sizeof(uint32_t) + 256 * (tiles + 1) * sizeof(uint32_t) + 256;
}

hipError_t launch_index(const float* mass, const float* cost, const int32_t* prompt_len,
                        const double* bin_repr, const int32_t* generated, int bucket, int Q, int B,
                        float* index, int32_t* argmin, hipStream_t stream, const IndexVariant* variant) {
  if (Q == 0) return hipSuccess;
  LaunchScope scope(variant ? (variant->levels > 0 ? "index_attained_table" : "index_variant")
                            : (generated ? "index_attained" : "index_scan"),
                    stream);
#define SAGE_INDEX_C(CC, GG) \
  return launch_index_c<CC, GG>(mass, cost, prompt_len, bin_repr, generated, bucket, Q, B, index, argmin, stream, \
                                variant)
  if (B <= 16) SAGE_INDEX_C(1, 16);
  if (B <= 32) SAGE_INDEX_C(2, 16);
  if (B <= 64) SAGE_INDEX_C(4, 16);
  if (B <= 128) SAGE_INDEX_C(8, 16);
  if (B <= 256) SAGE_INDEX_C(16, 16);
  if (B <= 512) SAGE_INDEX_C(16, 32);
  if (B <= 1024) SAGE_INDEX_C(16, 64);
  if (B <= 2048) SAGE_INDEX_C(32, 64);
  SAGE_INDEX_C(64, 64);
#undef SAGE_INDEX_C
}

hipError_t launch_rank(const float* index, int Q, int32_t* order, void* ws, hipStream_t stream) {
  if (Q == 0) return hipSuccess;
  if (Q <= kRankSmallMax) {
    // Requests per workgroup: the fewest that still leave >= 256 workgroups
    // (one per CU), so small queues spread over the chip.
    LaunchScope scope("rank_small", stream);
    if (Q <= 4096)
      hipLaunchKernelGGL(rank_count_kernel<16>, dim3((Q + 15) / 16), dim3(kRankCountThreads), 0, stream, index, Q, order);
    else
      hipLaunchKernelGGL(rank_count_kernel<32>, dim3((Q + 31) / 32), dim3(kRankCountThreads), 0, stream, index, Q, order);
    return hipGetLastError();
  }
  if (Q <= kRankMergeMax) {
    // Tiles of 512 sort faster, tiles of 1,024 are half as many to search; more
    // requests per workgroup read the tiles less often, fewer give more
    // workgroups. <512, 128> / <1024, 256> / <1024, 512>: 20,011 requests
    // 11.6 / 14.5 / 15.8 us, 65,536 26.9 / 21.8 / 27.3, 131,072 78.9 / 50.8 / 44.9.
    if (Q <= 32768) launch_rank_merge<512, 128>(index, Q, order, ws, stream);
    else if (Q <= 81920) launch_rank_merge<1024, 256>(index, Q, order, ws, stream);
    else launch_rank_merge<1024, 512>(index, Q, order, ws, stream);
    return hipGetLastError();
  }
  const int n_tiles = (Q + kRankTile - 1) / kRankTile;
  uint32_t* kA = static_cast<uint32_t*>(ws);
  uint32_t* vA = kA + Q;
  uint32_t* kB = vA + Q;
  uint32_t* vB = kB + Q;
  uint32_t* hist = vB + Q;
  uint32_t* totals = hist + 256 * (size_t)n_tiles;
  const uint32_t* k_in = nullptr;
  const uint32_t* v_in = nullptr;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 8 * pass;
    const bool last = pass == 3;
    uint32_t* k_out = last ? nullptr : (pass % 2 == 0 ? kA : kB);
    uint32_t* v_out = last ? reinterpret_cast<uint32_t*>(order) : (pass % 2 == 0 ? vA : vB);
    {
      LaunchScope scope("rank_hist", stream);
      hipLaunchKernelGGL(rank_hist_kernel, dim3(n_tiles), dim3(kRankThreads), 0, stream, index, k_in,
                         Q, shift, n_tiles, hist);
    }
    {
      LaunchScope scope("rank_scan", stream);
      hipLaunchKernelGGL(rank_scan_kernel, dim3(256), dim3(256), 0, stream, hist, n_tiles, totals);
    }
    {
      LaunchScope scope("rank_scatter", stream);
      hipLaunchKernelGGL(rank_scatter_kernel, dim3(n_tiles), dim3(kRankThreads), 0, stream, index,
                         k_in, v_in, Q, shift, n_tiles, hist, totals, k_out, v_out);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_in = k_out;
    v_in = v_out;
  }
  return hipSuccess;
}

}  // namespace sage
