// Per-sample reduction over the packed layout, the Delta-IFD score (Sec. 3.2, Eq. 3 and Eq. 4), the policy-latency
// monitor of the appendix and the perplexity of a sample.
// Both are tiny next to the loss kernel; what matters here is exact bookkeeping and a fixed
// summation order (no floating-point atomics), so results are bitwise reproducible.
#include "npd_kd_gang.hpp"

namespace npd {

constexpr int kSegBlock = 256;

__global__ __launch_bounds__(kSegBlock) void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)kSegBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kSegBlock) p[i] = v;
}

// Sum (of a thread) and number (of its wave) of the scored positions of [b, e): thread t of TH adds positions b + t,
// b + t + TH, ... in order; `own` is called with every position.  What such a sum waits for is a chain of loads per position,
// so up to kSumAhead positions' masks and values are requested together (values of positions that are not scored are read
// and left out).  Measured (MI355X, in a graph): 4 samples of 8,192 positions 10.1 us one position at a time, 4.8 us so; 10
// samples of 819 3.4 / 3.0.  TWO: batches of two besides, for samples of one or two positions per thread (1,024 of 300 3.2, 3.5
// in a batch of eight, 2.7 so; 16 of 300 2.9 and 2.4; the more code costs the others 0 .. 0.1 us, 4,096 of them 0.15).
constexpr int kSumAhead = 8;
template <int TH, int N, class Own>
__device__ __forceinline__ void masked_sum_step(const float* __restrict__ x, const uint8_t* __restrict__ mask, int64_t p0,
                                                int64_t e, int tid, float& acc, int& n, Own own) {
  uint8_t m[N];
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t p = p0 + i * TH + tid;
    const int64_t q = p < e ? p : p0;  // (a position of the range, not counted)
    m[i] = mask[q];
    v[i] = x ? x[q] : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t p = p0 + i * TH + tid;
    const bool scored = p < e && m[i];
    if (p < e) own(p);
    if (scored) acc += v[i];
    n += (int)__popcll(__ballot(scored));  // of the wave
  }
}
template <int TH, bool TWO, class Own>
__device__ __forceinline__ void masked_sum(const float* __restrict__ x, const uint8_t* __restrict__ mask, int64_t b, int64_t e,
                                           int tid, float& acc, int& n, Own own) {
  int64_t p = b;
  for (; e - p > (TWO ? 2 : 1) * TH; p += kSumAhead * TH) masked_sum_step<TH, kSumAhead>(x, mask, p, e, tid, acc, n, own);
  if (TWO && e - p > TH)
    masked_sum_step<TH, 2>(x, mask, p, e, tid, acc, n, own);
  else if (p < e)
    masked_sum_step<TH, 1>(x, mask, p, e, tid, acc, n, own);
}

// One sample, by 256 threads of the workgroup (thread `tid` of them; `fred`, `ired`: their four words each).  All threads
// of the workgroup call it alike: it holds the workgroup's barriers.  `seg` < 0: no sample, only the barriers.
template <bool TWO>
__device__ __forceinline__ void reduce_segment(int64_t T, int seg, int tid, const float* __restrict__ x,
                                               const uint8_t* __restrict__ mask, const int32_t* __restrict__ cu,
                                               float* seg_sum, int32_t* seg_count, float* seg_mean,
                                               int32_t* token_to_sample, int32_t* status, float* fred, int* ired) {
  constexpr int NW = kSegBlock / kWave;
  int64_t b = 0, e = 0;
  bool bad = false;
  if (seg >= 0) {
    b = cu[seg];
    e = cu[seg + 1];
    bad = b < 0 || e < b || e > T;
    if (bad) e = b;
  }
  float acc = 0.0f;
  int n = 0;
  masked_sum<kSegBlock, TWO>(x, mask, b, e, tid, acc, n, [&](int64_t p) {
    if (token_to_sample) token_to_sample[p] = seg;
  });
  // the 256 partials are folded by a fixed tree, the four wave totals in wave order
  acc = wave_sum_dpp(acc);
  if ((tid & (kWave - 1)) == 0) {
    fred[tid / kWave] = acc;
    ired[tid / kWave] = n;
  }
  __syncthreads();
  if (tid == 0 && seg >= 0) {
    acc = fred[0];
    n = ired[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      acc += fred[w];
      n += ired[w];
    }
    const float nanv = __builtin_nanf("");
    if (seg_sum) seg_sum[seg] = bad ? nanv : acc;
    if (seg_count) seg_count[seg] = bad ? 0 : n;
    if (seg_mean) seg_mean[seg] = bad ? nanv : (n > 0 ? acc / (float)n : 0.0f);
    if (bad && status) atomicOr(status, 4);  // NPD_DEV_BAD_CU_SEQLENS
  }
}

// One workgroup per sample.
__global__ __launch_bounds__(kSegBlock) void segment_reduce_kernel(int64_t T, const float* __restrict__ x,
                                                                   const uint8_t* __restrict__ mask,
                                                                   const int32_t* __restrict__ cu, float* seg_sum,
                                                                   int32_t* seg_count, float* seg_mean,
                                                                   int32_t* token_to_sample, int32_t* status) {
  __shared__ float fred[kSegBlock / kWave];
  __shared__ int ired[kSegBlock / kWave];
  reduce_segment<true>(T, blockIdx.x, threadIdx.x, x, mask, cu, seg_sum, seg_count, seg_mean, token_to_sample, status, fred, ired);
}

hipError_t launch_segment_reduce(int64_t T, int32_t S, const float* values, const uint8_t* mask, const int32_t* cu,
                                 float* seg_sum, int32_t* seg_count, float* seg_mean, int32_t* token_to_sample,
                                 int32_t* status, hipStream_t stream) {
  if (token_to_sample && T > 0) {
    const int64_t want = (T + kSegBlock - 1) / kSegBlock;
    const unsigned blocks = (unsigned)(want < 4096 ? want : 4096);
    const hipError_t e = launch_kernel(fill_i32_kernel, dim3(blocks), dim3(kSegBlock), 0, stream, token_to_sample, T, -1);
    if (e != hipSuccess) return e;
  }
  if (S > 0) {
    return launch_kernel(segment_reduce_kernel, dim3((unsigned)S), dim3(kSegBlock), 0, stream, T, values, mask, cu,
                         seg_sum, seg_count, seg_mean, token_to_sample, status);
  }
  return hipSuccess;
}

// One thread per pair.  The number of kept pairs is an integer sum: exact in any order.  ALONE: one workgroup takes all
// pairs and writes their number, which needs no launch in front that clears it
// (MI355X, in a graph: 4.4 us with that launch, 2.7 us so).
constexpr int kIfdAlone = 1024;
template <int BLOCK, bool ALONE>
__global__ __launch_bounds__(BLOCK) void delta_ifd_kernel(int32_t P, int32_t S, const float* __restrict__ ms,
                                                              const float* __restrict__ mt,
                                                              const int32_t* __restrict__ cnt,
                                                              const int32_t* __restrict__ pc,
                                                              const int32_t* __restrict__ pu, float lo, float hi,
                                                              uint32_t flags, float* ifd_s, float* ifd_t, float* delta,
                                                              uint8_t* zone, uint8_t* keep, int32_t* keep_count) {
  __shared__ int ired[BLOCK / kWave];
  int kept = 0;
  for (int64_t j = blockIdx.x * (int64_t)BLOCK + threadIdx.x; j < P; j += (int64_t)gridDim.x * BLOCK) {
    const int ic = pc[j], iu = pu[j];
    const float nanv = __builtin_nanf("");
    float fs = nanv, ft = nanv, d = nanv;
    uint8_t z = 3, kp = 0;  // NPD_ZONE_INVALID
    // a pair with an empty sample, a zero denominator or a mean loss that is not finite has no score (also where
    // plain division would give a finite ratio: 1 / inf = 0)
    if ((unsigned)ic < (unsigned)S && (unsigned)iu < (unsigned)S && cnt[ic] > 0 && cnt[iu] > 0 && ms[iu] != 0.0f &&
        mt[iu] != 0.0f && isfinite(ms[ic]) && isfinite(ms[iu]) && isfinite(mt[ic]) && isfinite(mt[iu])) {
      fs = ms[ic] / ms[iu];  // IEEE division
      ft = mt[ic] / mt[iu];
      d = ft - fs;
    }
    if (isfinite(fs) && isfinite(ft) && isfinite(d)) {
      z = d < lo ? 0 : (d > hi ? 2 : 1);
      kp = z == 1;
      if ((flags & 1u) && !(ft <= 1.0f)) kp = 0;
    } else {
      fs = ft = d = nanv;
    }
    if (ifd_s) ifd_s[j] = fs;
    if (ifd_t) ifd_t[j] = ft;
    if (delta) delta[j] = d;
    if (zone) zone[j] = z;
    if (keep) keep[j] = kp;
    kept += kp;
  }
  kept = block_sum_int<BLOCK>(kept, ired);
  if (threadIdx.x == 0 && keep_count) {
    if constexpr (ALONE)
      *keep_count = kept;
    else if (kept)
      atomicAdd(keep_count, kept);
  }
}

hipError_t launch_delta_ifd(int32_t P, int32_t S, const float* ms, const float* mt, const int32_t* cnt,
                            const int32_t* pc, const int32_t* pu, float lo, float hi, uint32_t flags, float* ifd_s,
                            float* ifd_t, float* delta, uint8_t* zone, uint8_t* keep, int32_t* keep_count,
                            hipStream_t stream) {
  // (nothing to clear without a count: 600 and 1,024 pairs 2.8 us by workgroups of 256, 2.9 and 3.0 us by one)
  if (P > 0 && P <= (keep_count ? kIfdAlone : kSegBlock)) {
    if (P <= kSegBlock)
      return launch_kernel(delta_ifd_kernel<kSegBlock, true>, dim3(1), dim3(kSegBlock), 0, stream, P, S, ms, mt, cnt, pc, pu,
                           lo, hi, flags, ifd_s, ifd_t, delta, zone, keep, keep_count);
    return launch_kernel(delta_ifd_kernel<kIfdAlone, true>, dim3(1), dim3(kIfdAlone), 0, stream, P, S, ms, mt, cnt, pc, pu,
                         lo, hi, flags, ifd_s, ifd_t, delta, zone, keep, keep_count);
  }
  if (keep_count) {
    const hipError_t e = launch_kernel(fill_i32_kernel, dim3(1), dim3(kSegBlock), 0, stream, keep_count, (int64_t)1, 0);
    if (e != hipSuccess) return e;
  }
  if (P > 0) {
    const int want = (P + kSegBlock - 1) / kSegBlock;
    const unsigned blocks = (unsigned)(want < 1024 ? want : 1024);
    return launch_kernel(delta_ifd_kernel<kSegBlock, false>, dim3(blocks), dim3(kSegBlock), 0, stream, P, S, ms, mt, cnt, pc, pu, lo, hi,
                         flags, ifd_s, ifd_t, delta, zone, keep, keep_count);
  }
  return hipSuccess;
}

// ---- policy-latency monitor (appendix, "Analysis of Policy Latency") and perplexity

constexpr int kLagBlock = 1024;

// Workgroup 0: the step's D_KL(learner || generator), the mean of kl_tok over the scored positions that a sample owns --
// with a valid cu_seqlens those are the scored positions of [cu[0], cu[S]) -- against the near-policy bound epsilon.
// Thread t adds positions begin + t, begin + t + 1024, ... in order, then one fixed tree: reproducible.
// Workgroups 1 ..: the means of four samples each, if they are wanted.  Both in one launch: the sums do not depend on one
// another, and each by itself is a few microseconds of waiting (MI355X, in a graph, two launches and one position at a
// time / this: 64 positions 5.5 / 2.7 us, 8,192 8.1 / 3.5, 32,768 20.5 / 6.1).
__global__ __launch_bounds__(kLagBlock) void policy_lag_kernel(int64_t T, int32_t S, const float* __restrict__ kl,
                                                               const uint8_t* __restrict__ mask,
                                                               const int32_t* __restrict__ cu, float epsilon,
                                                               float* seg_mean, int32_t* seg_count, float* batch_mean,
                                                               int32_t* batch_count, int32_t* exceeded, int32_t* status) {
  __shared__ float fred[kLagBlock / kWave];
  __shared__ int ired[kLagBlock / kWave];
  if (blockIdx.x > 0) {
    constexpr int NW = kSegBlock / kWave;
    const int sub = threadIdx.x / kSegBlock;
    const int64_t seg = (int64_t)(blockIdx.x - 1) * (kLagBlock / kSegBlock) + sub;
    reduce_segment<false>(T, seg < S ? (int)seg : -1, threadIdx.x % kSegBlock, kl, mask, cu, nullptr, seg_count, seg_mean, nullptr,
                   status, fred + sub * NW, ired + sub * NW);
    return;
  }
  int bad = 0;
  for (int i = threadIdx.x; i < S; i += kLagBlock)
    if (cu[i] > cu[i + 1]) bad = 1;
  if (S > 0 && threadIdx.x == 0 && (cu[0] < 0 || cu[S] > T)) bad = 1;
  bad = __syncthreads_or(bad);
  float acc = 0.0f;
  int n = 0;
  if (!bad && S > 0) masked_sum<kLagBlock, false>(kl, mask, cu[0], cu[S], threadIdx.x, acc, n, [](int64_t) {});
  constexpr int NW = kLagBlock / kWave;
  const int lane = threadIdx.x % kWave;
  acc = wave_sum_dpp(acc);
  if (lane == 0) {
    fred[threadIdx.x / kWave] = acc;
    ired[threadIdx.x / kWave] = n;
  }
  __syncthreads();
  acc = wave_sum_dpp<merge_lanes(NW)>(lane < NW ? fred[lane] : 0.0f);
  n = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) n += ired[w];
  if (threadIdx.x == 0) {
    const float mean = bad ? __builtin_nanf("") : (n > 0 ? acc / (float)n : 0.0f);
    if (batch_mean) *batch_mean = mean;
    if (batch_count) *batch_count = bad ? 0 : n;
    if (exceeded) *exceeded = !(mean <= epsilon);  // near-policy: D_KL <= epsilon; NaN counts as beyond
    if (bad && status) atomicOr(status, 4);        // NPD_DEV_BAD_CU_SEQLENS
  }
}

hipError_t launch_policy_lag(int64_t T, int32_t S, const float* kl, const uint8_t* mask, const int32_t* cu,
                             float epsilon, float* seg_mean, int32_t* seg_count, float* batch_mean,
                             int32_t* batch_count, int32_t* exceeded, int32_t* status, hipStream_t stream) {
  constexpr int kSegs = kLagBlock / kSegBlock;
  int64_t seg_blocks = S > 0 && (seg_mean || seg_count) ? ((int64_t)S + kSegs - 1) / kSegs : 0;
  // a grid has fewer than 2^32 threads: the last few numbers of samples that a launch of their own takes (2^24 - 1 of 256
  // threads) leave no room for workgroup 0
  if ((1 + seg_blocks) * kLagBlock > 0xffffffffLL) {
    seg_blocks = 0;
    const hipError_t e = launch_segment_reduce(T, S, kl, mask, cu, nullptr, seg_count, seg_mean, nullptr, status, stream);
    if (e != hipSuccess) return e;
  }
  return launch_kernel(policy_lag_kernel, dim3((unsigned)(1 + seg_blocks)), dim3(kLagBlock), 0, stream, T, S, kl, mask, cu,
                       epsilon, seg_mean, seg_count, batch_mean, batch_count, exceeded, status);
}

// PPL = exp(mean CE loss) of every sample; 0 for samples without a scored position
__global__ __launch_bounds__(kSegBlock) void segment_ppl_kernel(int32_t S, const float* __restrict__ mean_nll,
                                                                const int32_t* __restrict__ cnt, float* ppl) {
  for (int64_t i = blockIdx.x * (int64_t)kSegBlock + threadIdx.x; i < S; i += (int64_t)gridDim.x * kSegBlock)
    ppl[i] = cnt[i] > 0 ? expf(mean_nll[i]) : 0.0f;
}

hipError_t launch_segment_ppl(int32_t S, const float* mean_nll, const int32_t* cnt, float* ppl, hipStream_t stream) {
  if (S <= 0) return hipSuccess;
  const int want = (S + kSegBlock - 1) / kSegBlock;
  return launch_kernel(segment_ppl_kernel, dim3((unsigned)(want < 1024 ? want : 1024)), dim3(kSegBlock), 0, stream, S,
                       mean_nll, cnt, ppl);
}

}  // namespace npd
