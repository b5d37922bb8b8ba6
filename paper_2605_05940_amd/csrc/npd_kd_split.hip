// Forward-only calls whose rows are split over several workgroups: a workgroup of 256 threads sums one slice of a row and
// leaves its partial log-sum-exps in a scratch record; a second kernel, a wave to a row, merges a row's partials and writes
// its scalars.
//
// Why: with a workgroup per row a row takes as long as one compute unit needs for it, which is its vector instructions
// (17 us for the 151,936 pairs of logits of a dense teacher) behind the latency of its first loads; rows that are
// fewer than the compute units leave the others idle, and the last rows of many leave most of them idle.  A slice is read,
// summed once and gone; with two launches nothing waits for another workgroup.  The second launch costs about 2.5 us: calls of few
// rows on a kept record whose words carry the launch's number (KdArgs::tag, npd_kd_gang.hpp) have none, there the last slice of a
// row waits for the others' partials and merges them (forward progress and bounded waits as in npd_kd_gang.hpp).
#include "npd_kd_gang.hpp"

namespace npd {

namespace {

constexpr int kSplitThreads = 256;
constexpr int kSplitMax = kWave;  // slices per row at most: a lane each in the second kernel

// partial log-sum-exps: 0 student / tau, 1 teacher / tau with the cross term, 2 student and 3 teacher at tau = 1 (LSE1); no
// teacher: the student's at tau = 1 alone
constexpr int split_sums(bool dense, bool lse1) { return dense ? (lse1 ? 4 : 2) : 1; }
constexpr int split_words(bool dense, bool lse1) { return split_sums(dense, lse1) * 3; }

}  // namespace

// A row's scalars from its totals (one lane).
template <bool DENSE, bool LSE1>
__device__ __forceinline__ void split_row_scalars(const KdArgs& a, int64_t row, int y, float s_y, float t_y,
                                                  Lse (&acc)[split_sums(DENSE, LSE1)], bool timeout) {
  constexpr int NS = split_sums(DENSE, LSE1);
  const float nanv = __builtin_nanf("");
  const float Ls = acc[0].log2_sum();
  const float lse1_s = timeout ? nanv : __fmul_rn(LSE1 ? acc[NS == 4 ? 2 : 0].log2_sum() : Ls, kLn2);
  float lse1_t = 0.0f;
  if constexpr (DENSE) {
    lse1_t = timeout ? nanv : __fmul_rn(LSE1 ? acc[NS == 4 ? 3 : 1].log2_sum() : acc[1].log2_sum(), kLn2);
    const float lse_diff = ((acc[0].r - acc[1].r) + (acc[0].log2_z() - acc[1].log2_z())) * kLn2;  // lse_S - lse_T at tau
    const float kd = (acc[1].a / acc[1].z) * a.inv_tau + lse_diff;
    if (a.kd) a.kd[row] = timeout ? nanv : kd < 0.0f ? 0.0f : kd;
  }
  if (a.lse) a.lse[row] = lse1_s;
  const bool bad_label = a.labels && (unsigned)y >= (unsigned)a.V;
  if (a.nll) a.nll[row] = bad_label ? nanv : __fsub_rn(lse1_s, s_y);
  if (a.tnll) a.tnll[row] = bad_label ? nanv : __fsub_rn(lse1_t, t_y);
  int flags = timeout ? 8 : 0;                            // NPD_DEV_GANG_TIMEOUT
  if (bad_label && (a.nll || a.tnll)) flags |= 1;         // NPD_DEV_BAD_LABEL
  if (flags && a.status) atomicOr(a.status, flags);
}
__device__ __forceinline__ void split_row_zeros(const KdArgs& a, int64_t row) {
  if (a.kd) a.kd[row] = 0.0f;
  if (a.nll) a.nll[row] = 0.0f;
  if (a.tnll) a.tnll[row] = 0.0f;
  if (a.lse) a.lse[row] = 0.0f;
}

// K: groups per thread and tensor; a slice is a.gang_groups <= K * 256 groups long.  ONE: the only launch of the call.
template <int K, bool DENSE, bool LSE1, bool ONE>
__global__ __launch_bounds__(kSplitThreads, 4) void kd_split_kernel(const KdArgs a) {
  constexpr int TH = kSplitThreads, GB = TH * 16, NS = split_sums(DENSE, LSE1), W = split_words(DENSE, LSE1);
  constexpr int NWV = TH / kWave;
  __shared__ float red[NS * 3 * NWV];
  __shared__ uint32_t xch[ONE ? kSplitMax * W : 1];
  __shared__ int gave_up;
  const int G = a.gang;
  const int64_t row = blockIdx.x / (unsigned)G;
  const int slice = (int)(blockIdx.x - (unsigned)(row * G));
  const bool merges = ONE && slice == G - 1;  // uniform
  if (!a.mask[row]) {  // (the second kernel writes its zeros, where there is one)
    if (merges && threadIdx.x == 0) split_row_zeros(a, row);
    return;
  }
  if (ONE && threadIdx.x == 0) gave_up = 0;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  const int V = a.V;
  const uint16_t* srow = a.s + row * a.s_stride;
  const uint16_t* trow = DENSE ? a.t + row * a.t_stride : nullptr;
  const RowSplit sp = row_split(srow, V, true);
  const int head = sp.head, nvec = sp.nvec, n_edge = V - nvec * 8;
  const int b0 = slice * a.gang_groups, b1 = b0 + a.gang_groups;
  const int g0 = b0 < nvec ? b0 : nvec, g1 = slice == G - 1 ? nvec : (b1 < nvec ? b1 : nvec);
  const int ng = g1 - g0;
  const float c = DENSE ? a.c : kLog2e;
  const bool lse1_t = LSE1 && a.tnll != nullptr;

  const __amdgpu_buffer_rsrc_t rs = row_rsrc(srow + head + (size_t)g0 * 8, ng);
  const __amdgpu_buffer_rsrc_t rt = row_rsrc((DENSE ? trow : srow) + head + (size_t)g0 * 8, ng);
  const int voff = tid * 16;
  const int n_mine = (ng - tid + TH - 1) / TH;  // groups of this thread
  uint4 sreg[K], treg[DENSE ? K : 1];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    sreg[k] = ld_group<GB>(rs, voff, k, true, true);
    if constexpr (DENSE) treg[k] = ld_group<GB>(rt, voff, k, true, true);
  }
  int y = -1;
  uint32_t s_y = 0, t_y = 0;
  if (merges && a.labels) {
    y = a.labels[row];
    if ((unsigned)y < (unsigned)V) {
      s_y = srow[y];
      if constexpr (DENSE) t_y = trow[y];
    }
  }
  Lse acc[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) acc[i].init();
  __builtin_amdgcn_sched_barrier(0);

  // As in kd_gang_kernel: every thread's references are the largest of its logits, no element is inspected again, and a wave
  // whose sums show something else (a logit of -inf in the cross term) sums its registers once more in the careful form.
  if (ng > tid) {
    const float fs = thread_max(sreg, n_mine);
    acc[0].r = __builtin_rintf(__builtin_fmaxf(fs * c, -1.0e30f));
    if constexpr (LSE1) acc[2].r = __builtin_rintf(__builtin_fmaxf(fs * kLog2e, -1.0e30f));
    if constexpr (DENSE) {
      const float ft = thread_max(treg, n_mine);
      acc[1].r = __builtin_rintf(__builtin_fmaxf(ft * c, -1.0e30f));
      if constexpr (LSE1) acc[3].r = __builtin_rintf(__builtin_fmaxf(ft * kLog2e, -1.0e30f));
    }
  }
  // A dense teacher's logits are unpacked, and subtracted, by the matrix cores (a logit that is not finite shows in the sums):
  // 6,000 rows of 151,936 549 / 533 us, at tau = 2 with NLLs 652 / 633; of 50,304 177 / 180, 225 / 218.
  const s16x4 identity = lane_identity(kBf16One);
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
#pragma unroll
  for (int k = 0; k < K; ++k) {
    float xs[8], xt[8], d[8];
    if constexpr (DENSE) {
      if (k * TH + wave0 >= ng) break;  // uniform: no group for this wave from here on
      unpack8_mfma(sreg[k], identity, xs);
      unpack8_mfma(treg[k], identity, xt);
      mfma8(sreg[k], identity ^ (short)0x8000, xt, d);
    }
    if (k < n_mine) {
      if constexpr (!DENSE) unpack8(sreg[k], xs);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        acc[0].z += exp2_fast(__builtin_fmaf(xs[j], c, -acc[0].r));
        if constexpr (DENSE) {
          const float et = exp2_fast(__builtin_fmaf(xt[j], c, -acc[1].r));
          acc[1].z += et;
          acc[1].a = __builtin_fmaf(et, d[j], acc[1].a);
        }
        if constexpr (LSE1) {
          acc[2].z += exp2_fast(__builtin_fmaf(xs[j], kLog2e, -acc[2].r));
          if (lse1_t) acc[3].z += exp2_fast(__builtin_fmaf(xt[j], kLog2e, -acc[3].r));
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  {
    constexpr float kBig = 1.2676506e30f;  // 2^100
    bool odd = false;
#pragma unroll
    for (int i = 0; i < NS; ++i) odd = odd || !(acc[i].z < kBig) || !(fabsf(acc[i].a) < kBig);
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {  // wave-uniform
#pragma unroll
      for (int i = 0; i < NS; ++i) acc[i].init();
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (k < n_mine) {
          if constexpr (DENSE) {
            accum8<kDense, LSE1, false>(sreg[k], treg[k], c, lse1_t, acc);
          } else {
            float xs[8];
            unpack8(sreg[k], xs);
            acc[0].add8(xs, c);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (slice == G - 1 && tid < n_edge) {
    const int e = sp.edge_elem(tid);
    const float xs = bf16_one(srow[e]);
    acc[0].add1(xs, c);
    if constexpr (LSE1) acc[2].add1(xs, kLog2e);
    if constexpr (DENSE) {
      const float xt = bf16_one(trow[e]);
      acc[1].add1_cross(xt, xt - xs, c);
      if constexpr (LSE1)
        if (lse1_t) acc[3].add1(xt, kLog2e);
    }
  }

  // ---- wave totals, workgroup totals, left in the record
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    normalise(acc[i]);
    wave_merge_rescaled<true>(acc[i]);
    if (lane == 0) {
      red[(i * 3 + 0) * NWV + wid] = acc[i].r;
      red[(i * 3 + 1) * NWV + wid] = acc[i].z;
      red[(i * 3 + 2) * NWV + wid] = acc[i].a;
    }
  }
  __syncthreads();
  if (!merges && wid > 0) return;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    acc[i].init();
    if (lane < NWV) {
      acc[i].r = red[(i * 3 + 0) * NWV + lane];
      acc[i].z = red[(i * 3 + 1) * NWV + lane];
      acc[i].a = red[(i * 3 + 2) * NWV + lane];
    }
    wave_merge_rescaled<true, merge_lanes(NWV)>(acc[i]);
  }
  if constexpr (!ONE) {
    if (lane == 0) {
      float* rec = reinterpret_cast<float*>(a.ws) + (size_t)blockIdx.x * W;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        rec[i * 3 + 0] = acc[i].r;
        rec[i * 3 + 1] = acc[i].z;
        rec[i * 3 + 2] = acc[i].a;
      }
    }
  } else {
    float v = acc[0].r;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      if (lane == i * 3 + 0) v = acc[i].r;
      if (lane == i * 3 + 1) v = acc[i].z;
      if (lane == i * 3 + 2) v = acc[i].a;
    }
    if (!merges) {
      if (lane < W) gang_post(a.ws, (size_t)blockIdx.x * W + lane, v, a.tag);
      return;
    }
    if (wid == 0 && lane < W) xch[slice * W + lane] = __builtin_bit_cast(uint32_t, v);
    for (int w = tid; w < slice * W; w += TH)
      xch[w] = gang_wait(a.ws, (size_t)row * G * W + w, (size_t)gridDim.x * W, a.tag, a.spin_limit, &gave_up);
    __syncthreads();
    if (wid > 0) return;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      acc[i].init();
      if (lane < G) {
        acc[i].r = __builtin_bit_cast(float, xch[lane * W + i * 3 + 0]);
        acc[i].z = __builtin_bit_cast(float, xch[lane * W + i * 3 + 1]);
        acc[i].a = __builtin_bit_cast(float, xch[lane * W + i * 3 + 2]);
      }
      wave_merge_rescaled<true>(acc[i]);
    }
    if (lane == 0) split_row_scalars<DENSE, LSE1>(a, row, y, bf16_lo(s_y), bf16_lo(t_y), acc, gave_up != 0);
  }
}

// Four rows to a workgroup, a wave each.
template <bool DENSE, bool LSE1>
__global__ __launch_bounds__(kSplitThreads) void kd_split_merge_kernel(const KdArgs a) {
  constexpr int NS = split_sums(DENSE, LSE1), W = split_words(DENSE, LSE1);
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t row = (int64_t)blockIdx.x * (kSplitThreads / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (row >= a.T) return;
  if (!a.mask[row]) {
    if (lane == 0) split_row_zeros(a, row);
    return;
  }
  int y = -1;
  float s_y = 0.0f, t_y = 0.0f;
  if (a.labels) {
    y = a.labels[row];
    if ((unsigned)y < (unsigned)a.V) {
      s_y = bf16_one(a.s[row * a.s_stride + y]);
      if constexpr (DENSE) t_y = bf16_one(a.t[row * a.t_stride + y]);
    }
  }
  const float* rec = reinterpret_cast<const float*>(a.ws) + ((size_t)row * a.gang + lane) * W;
  Lse acc[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    acc[i].init();
    if (lane < a.gang) {
      acc[i].r = rec[i * 3 + 0];
      acc[i].z = rec[i * 3 + 1];
      acc[i].a = rec[i * 3 + 2];
    }
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) wave_merge_rescaled<true>(acc[i]);
  if (lane == 0) split_row_scalars<DENSE, LSE1>(a, row, y, s_y, t_y, acc, false);
}

namespace {

// Groups per thread, 0: not split.  Four groups of a dense teacher for few rows, eight for many (2,048 rows of 151,936 at tau
// = 2: 246 / 225 us).  Measured (MI355X, all scored, us, a workgroup per row / split; the dense kernel with a workgroup per row
// runs two rows to a compute unit, so its time steps up behind every multiple of 512 rows):
//   dense teacher, tau = 1   1 row of 151,936 20.0 / 6.7;  64 rows of 50,304 10.0 / 7.8, 151,936 21.1 / 11.9;  181 rows of
//                            151,936 22.9 / 21.4;  256 rows of 50,304 12.1 / 13.1, 131,072 and more the same or less;  257 rows
//                            of 50,304 16.3 / 14.8, 400 18.6 / 18.5, 440 .958 of the speed at 60,000, 512 19.8 / 21.3, 520
//                            1.15, 700 .99 .. 1.06, 768 .974 .. 1.05, 800 32.3 / 29.5;  512 of 100,352 36.1 / 35.3;  6,000 rows of
//                            50,304 182 / 182, 151,936 541 / 510  (32,000: 128 rows 8.4 / 8.2, 4,096 80.7 / 84.2)
//   dense teacher, tau = 2, both NLLs    128 rows of 151,936 33.4 / 23.2;  512 of 50,304 1.06;  6,000 rows of 50,304 255 / 218,
//                            151,936 792 / 633
//   the student's alone (speed; the other kernel then has less to do, this one as many instructions)   50,304: 512 rows .971,
//                            600 1.09, 1,024 .98, 1,400 1.04, 1,536 .973, 6,000 .95;  100,352 512 1.02, 1,024 .96, 1,400 1.01, 6,000 .90;
//                            41,000 6,000 1.05;  110,000 512 1.23, 6,000 1.34
//   no teacher               64 rows of 65,536 6.9 / 6.2, of 75,000 .952, of 90,000 1.06;  100 rows of 100,352 1.02, 112 .932, 128
//                            8.7 / 9.6, of 116,000 1.03;  128 rows of 151,936 12.3 / 11.0;  240,000: 130 .. 256 rows .95 .. .98, 300
//                            1.26, 500 .. 1,024 .97 .. .99, 2,000 1.02;  262,144: 181 rows 20.4 / 19.3, 256 .995, 1,000 .996, 4,096
//                            339 / 323  (181 rows of 151,936 11.7 / 13.4, 1,024 of 200,000 63.9 / 66.1)
enum Tau1Sums { kNoSums, kStudentSum, kBothSums };  // at tau = 1, beside others
int split_groups(int64_t T, int nvec, bool dense, Tau1Sums sums) {
  constexpr int kFew = 256;  // rows: one to a compute unit
  if (dense) {
    if (nvec <= 5120 || (T > kFew / 2 && T <= kFew && nvec < 16384)) return 0;
    if (sums != kBothSums && T > 432 && T <= 2 * kFew && nvec < 12288) return 0;
    if (sums == kStudentSum && (T > 1400 || (T > 960 && T <= 4 * kFew)) && nvec >= 5500 && nvec < 13000) return 0;
    return T <= kFew ? 4 : 8;
  }
  if (nvec >= 32768) return 8;
  if (nvec >= 30000) return T <= kFew / 2 || (T > kFew && T <= 448) || T > 1024 ? 8 : 0;
  if (nvec >= 12288) return T <= 104 || (T <= kFew / 2 && nvec >= 14500) ? 8 : 0;
  return nvec >= 8192 && T <= (nvec > 10240 ? 64 : 51) ? 8 : 0;
}

// Rows up to which a call on a kept record is one launch: a workgroup that waits keeps its place on a compute unit from the
// slices behind it, and the second launch counts for less the longer the first is.  Measured (MI355X, us of the loss and the
// monitor's reduction, dense teacher, seven tenths scored, two launches / one): 16 rows of 151,936 12.2 / 9.9, 256 25.6 / 24.1,
// 64 of 50,304 12.1 / 9.8, 400 of 100,352 27.6 / 26.2;  700 of 151,936 51.6 / 52.1, 5,000 305 / 311, of 50,304 112 / 121.
constexpr int64_t kSplitOneLaunchRows = 512;

// slices of a row of nvec groups, 0: not split
int split_slices(int64_t T, int nvec, bool dense, Tau1Sums sums) {
  const int cap = split_groups(T, nvec, dense, sums) * kSplitThreads;
  if (cap == 0) return 0;
  const int g = (nvec + cap - 1) / cap;
  return g >= 2 && g <= kSplitMax && T * (int64_t)g <= 0x7fffffffLL ? g : 0;
}

template <int K, bool DENSE, bool LSE1>
hipError_t launch_split(const KdArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)(a.T * a.gang));
  if (a.tag != 0) return launch_kernel(kd_split_kernel<K, DENSE, LSE1, true>, grid, dim3(kSplitThreads), 0, stream, a);
  const hipError_t e = launch_kernel(kd_split_kernel<K, DENSE, LSE1, false>, grid, dim3(kSplitThreads), 0, stream, a);
  if (e != hipSuccess) return e;
  constexpr int rows = kSplitThreads / kWave;
  return launch_kernel(kd_split_merge_kernel<DENSE, LSE1>, dim3((unsigned)((a.T + rows - 1) / rows)), dim3(kSplitThreads), 0,
                       stream, a);
}

}  // namespace

size_t split_scratch_bytes(int64_t T, int32_t V, int teacher_kind, int divergence, bool lse1) {
  if ((teacher_kind != kDense && teacher_kind != kNone) || divergence != kForwardKl) return 0;
  const bool dense = teacher_kind == kDense;
  const int g = split_slices(T, V / 8, dense, dense && lse1 ? kBothSums : kNoSums);  // (split if any of them is)
  return (size_t)T * g * split_words(dense, dense && lse1) * sizeof(float);
}

size_t split_kept_bytes(int64_t T, size_t scratch_bytes) {
  return T <= kSplitOneLaunchRows && scratch_bytes > 0 ? 2 * (scratch_bytes + kGangTailWords * sizeof(uint32_t)) : 0;
}

static Tau1Sums tau1_sums(const KdArgs& a, bool dense) {
  return !dense || !a.need_lse1 ? kNoSums : a.tnll ? kBothSums : kStudentSum;
}
bool split_path_applies(const KdArgs& a, int teacher_kind) {
  const bool dense = teacher_kind == kDense;
  return split_slices(a.T, a.nvec_s, dense, tau1_sums(a, dense)) > 0;
}

hipError_t launch_kd_split(const KdArgs& a0, int teacher_kind, hipStream_t stream) {
  KdArgs a = a0;
  const bool dense = teacher_kind == kDense;
  a.gang = split_slices(a.T, a.nvec_s, dense, tau1_sums(a, dense));
  a.gang_groups = ((a.nvec_s + a.gang - 1) / a.gang + 7) / 8 * 8;
  a.spin_limit = gang_spin_limit();
  if (!dense) return launch_split<8, false, false>(a, stream);
  if (split_groups(a.T, a.nvec_s, true, tau1_sums(a, true)) == 4)
    return a.need_lse1 ? launch_split<4, true, true>(a, stream) : launch_split<4, true, false>(a, stream);
  return a.need_lse1 ? launch_split<8, true, true>(a, stream) : launch_split<8, true, false>(a, stream);
}

}  // namespace npd
