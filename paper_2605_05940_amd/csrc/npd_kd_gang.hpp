// Row-gang variant of the fused KD loss + gradient kernel (gfx950): a token row is shared by G short-lived
// workgroups of 256 threads, each of which owns a slice of the row (up to K 128-bit groups per thread and tensor, in pieces
// of 4 KB that are dealt to the row's workgroups in turn) and keeps it in registers from the first sweep to the gradient write -- nothing is read twice, whatever
// the vocabulary.  The G partial log-sum-exps of a row meet through a small scratch record in device memory:
//
//   sweep 1 over the slice -> workgroup partials (r, z, a) -> posted to scratch[row][slice]
//   wait until all G slices of the row have posted -> merge them in one fixed tree (every workgroup of the row
//   computes bit-identical row totals) -> gradient of the slice from the registers -> written once
//
// Why: the memory system of this GPU gives a mix of two reads and one write 6.7 TB/s when the chip sweeps memory
// front to back, every row is read completely before it is written and no cache line is shared by two workgroups,
// against 5.7 TB/s when each compute unit works on a row of its own.  Consecutive workgroups take consecutive pieces
// (which begin on 128-byte boundaries of the row) and write them side by side, four workgroups run per compute unit (one row's wait and arithmetic
// overlap three other slices' memory traffic), and the workgroups of rows that are not scored zero-fill their slices
// in the same address order.
//
// The exchange needs no fence: every posted word is an atomic store that carries its own validity, and consumers poll those
// words with atomic loads at device scope.  Either the scratch record is cleared to a pattern no posted word takes, by a fill
// kernel enqueued in front of each launch, and words are 32 bits; or (KdArgs::tag) words are 64 bits, the upper half a number
// that no earlier launch on this record has had, and there is no launch in front (a record that was zero once and has been used
// by such launches alone; the fill and its gap take 2.4 us of a small call, 5 us of a large one).  Forward progress: a workgroup waits only for
// workgroups of smaller or neighbouring index (the other slices of its own row), a workgroup never waits before it
// has posted, and workgroups start in index order, so the lowest unfinished row always has all its workgroups
// resident or next to start.  Every wait is bounded all the same: a workgroup that gives up marks its row NaN, sets
// NPD_DEV_GANG_TIMEOUT and raises a launch-wide flag that ends every other wait of the launch early, so a kernel can
// never hang, nor spend one limit per row.
#pragma once
#include <type_traits>

#include "npd_kd_cached.hpp"

namespace npd {

constexpr int kGangThreads = 256;
constexpr int kGangMax = 32;                      // slices per row at most
constexpr uint32_t kGangEmpty = 0xffffffffu;      // scratch word not posted yet (a NaN pattern no partial is stored as)
constexpr int kGangSpinLimitDefault = 1 << 20;    // polls before a workgroup gives up (seconds; never reached in a healthy run)

// ---- merging partial log-sum-exps: largest reference first, every partial rescaled to it once, then plain sums.
// Cross-lane steps are DPP operands of the adds and maxima (no LDS traffic, no address arithmetic); the order of operations is
// fixed, so results are bitwise reproducible and two streams fed the same data stay bitwise identical.
__device__ __forceinline__ float lane63(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
__device__ __forceinline__ float lane0(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}
// Sum / maximum over the 64 lanes, every lane gets the result: pairs, quads, half rows, rows of 16, then lane 15 of
// rows 0 / 2 into rows 1 / 3 and lane 31 into rows 2 and 3, so that lane 63 holds everything.  Each step is one
// instruction whose first operand is read through DPP (lanes that a row mask leaves out keep their value); written out
// because the compiler spends four instructions per step on the maximum.  A DPP operand must not be read within two
// wait states of the instruction that wrote it: hence the s_nop in front of every step.
// LANES < 64: only the first LANES lanes hold something and lane 0 gives the result -- the same steps as far as they change
// it.
#define NPD_DPP_STEP(op, how) "s_nop 1\n" op " %0, %0, %0 " how "\n"
#define NPD_DPP_REDUCE4(op)                                                          \
  "s_nop 4\n" op " %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"      \
  NPD_DPP_STEP(op, "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
#define NPD_DPP_REDUCE16(op)                                                         \
  NPD_DPP_REDUCE4(op)                                                                \
  NPD_DPP_STEP(op, "row_half_mirror row_mask:0xf bank_mask:0xf")                     \
  NPD_DPP_STEP(op, "row_mirror row_mask:0xf bank_mask:0xf")
#define NPD_DPP_REDUCE(op)                                                           \
  NPD_DPP_REDUCE16(op)                                                               \
  NPD_DPP_STEP(op, "row_bcast:15 row_mask:0xa bank_mask:0xf")                        \
  NPD_DPP_STEP(op, "row_bcast:31 row_mask:0xc bank_mask:0xf")                        \
  "s_nop 1\n"
template <int LANES = kWave>
__device__ __forceinline__ float wave_sum_dpp(float x) {
  static_assert(LANES == 4 || LANES == 16 || LANES == kWave, "");
  if constexpr (LANES == 4)
    asm volatile(NPD_DPP_REDUCE4("v_add_f32_dpp") "s_nop 1\n" : "+v"(x));
  else if constexpr (LANES == 16)
    asm volatile(NPD_DPP_REDUCE16("v_add_f32_dpp") "s_nop 1\n" : "+v"(x));
  else
    asm volatile(NPD_DPP_REDUCE("v_add_f32_dpp") : "+v"(x));
  return LANES == kWave ? lane63(x) : lane0(x);
}
template <int LANES = kWave>
__device__ __forceinline__ float wave_max_dpp(float x) {
  if constexpr (LANES == 4)
    asm volatile(NPD_DPP_REDUCE4("v_max_f32_dpp") "s_nop 1\n" : "+v"(x));
  else if constexpr (LANES == 16)
    asm volatile(NPD_DPP_REDUCE16("v_max_f32_dpp") "s_nop 1\n" : "+v"(x));
  else
    asm volatile(NPD_DPP_REDUCE("v_max_f32_dpp") : "+v"(x));
  return LANES == kWave ? lane63(x) : lane0(x);
}
// merges the 64 lanes' partials (sum = z 2^r, cross term a 2^r); every lane returns with the total
template <bool CROSS, int LANES = kWave>
__device__ __forceinline__ void wave_merge_rescaled(Lse& v) {
  const float R = wave_max_dpp<LANES>(v.r);
  const float f = exp2_fast(v.r - R);  // exactly 1 where r == R; 0 for empty partials far below
  v.z = wave_sum_dpp<LANES>(__fmul_rn(v.z, f));
  if constexpr (CROSS) v.a = wave_sum_dpp<LANES>(__fmul_rn(v.a, f));
  v.r = R;
}
// the lanes that a merge of n partials goes through
constexpr int merge_lanes(int n) { return n <= 4 ? 4 : n <= 16 ? 16 : kWave; }
// a lane's partial with its sum brought into [1, 2): r takes up the exponent of z, so that later rescaling to a
// larger reference can only shrink values (z may be anywhere below 2^100 when the reference was a guess)
__device__ __forceinline__ void normalise(Lse& v) {
  const int e = (int)((__builtin_bit_cast(uint32_t, v.z) >> 23) & 0xffu) - 127;
  if (v.z > 0.0f && e > -127 && e < 128) {  // normal, positive (zero, NaN and infinity stay as they are)
    const float down = __builtin_bit_cast(float, (uint32_t)(127 - e) << 23);  // 2^-e
    v.z = __fmul_rn(v.z, down);
    v.a = __fmul_rn(v.a, down);
    v.r += (float)e;
  }
}

// Largest of the eight bf16 values packed in a group, as a float -- by packed 16-bit integer maxima on the bit
// patterns, which order non-negative values correctly and put every negative value below them.  Among negative
// values alone the integer order is the reverse of the value order, so for a group whose logits are all negative the
// result is its smallest logit: still a usable reference exponent (lower by the spread of the group), and the
// caller's check of the sums catches the case where that is not enough.
typedef short s16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max_i16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, a), __builtin_bit_cast(s16x2, b)));
}
__device__ __forceinline__ uint32_t pk_max_group(const uint4& v) { return pk_max_i16(pk_max_i16(v.x, v.y), pk_max_i16(v.z, v.w)); }
__device__ __forceinline__ float pk_max_value(uint32_t m) {
  const int lo = (int)(short)(m & 0xffffu), hi = (int)(short)(m >> 16);
  return bf16_one((uint16_t)(lo > hi ? lo : hi));
}

// Largest logit of a thread's groups (mine(k); at least one; FIRST: not always the first), whatever their signs, with v_pk_max_f16: fp16 patterns are sign and
// magnitude like bf16 ones, so their order is the same.  The patterns it takes for NaN are magnitudes of more than
// 2^121: infinities and NaN, which it passes over while the other operand is a number.  Where there is nothing else the
// result is far below every logit: sums against it are 0 if all logits are -inf and show an anomaly otherwise.  (Written
// out because the compiler canonicalises both operands of the builtin.)
__device__ __forceinline__ uint32_t pk_max_bf16(uint32_t a, uint32_t b) {
  uint32_t d;
  asm("v_pk_max_f16 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
template <bool FIRST, int K, class Mine>
__device__ __forceinline__ float thread_max(const uint4 (&v)[K], Mine mine) {
  constexpr uint32_t kNothing = 0xff80ff80u;  // a pair of -inf, for the groups that are not the thread's
  uint32_t m = kNothing;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint32_t g = pk_max_bf16(pk_max_bf16(v[k].x, v[k].y), pk_max_bf16(v[k].z, v[k].w));
    const uint32_t w = (k == 0 && !FIRST) || mine(k) ? g : kNothing;
    m = k == 0 ? w : pk_max_bf16(m, w);
  }
  const float lo = bf16_lo(m), hi = bf16_hi(m);
  const float x = lo > hi ? lo : hi;
  return fabsf(x) < 2.6e36f ? x : -3.0e38f;
}
// ... of its first n >= 1 groups
template <int K>
__device__ __forceinline__ float thread_max(const uint4 (&v)[K], int n) {
  return thread_max<false>(v, [&](int k) __attribute__((always_inline)) { return k < n; });
}

__device__ __forceinline__ void gang_post(uint32_t* ws, size_t at, float v, uint32_t tag) {
  uint32_t w = __builtin_bit_cast(uint32_t, v);
  if (tag != 0) {  // uniform
    __hip_atomic_store(reinterpret_cast<uint64_t*>(ws) + at, (uint64_t)tag << 32 | w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (w == kGangEmpty) w = 0x7fc00000u;  // another NaN
  __hip_atomic_store(ws + at, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits for posted word `at`.  Gives up after `spin_limit` polls, or -- looked at every 256th poll -- as soon as any
// workgroup of the launch has given up (word `abandon` behind the record, posted then): once one wait has run out, no
// other workgroup spends its own limit, so a launch whose workgroups cannot see each other ends within seconds
// however many rows it has.  Returns the word, or anything with *gave_up set.
constexpr int kGangTailWords = 64;  // words behind the record; word 0: a workgroup has given up
__device__ __forceinline__ bool gang_look(const uint32_t* ws, size_t at, uint32_t tag, uint32_t& w) {
  if (tag != 0) {  // uniform
    const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(ws) + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    w = (uint32_t)v;
    return (uint32_t)(v >> 32) == tag;
  }
  w = __hip_atomic_load(ws + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return w != kGangEmpty;
}
__device__ __forceinline__ uint32_t gang_wait(uint32_t* ws, size_t at, size_t abandon, uint32_t tag, int spin_limit, int* gave_up) {
  int spins = 0;
  while (true) {
    uint32_t w, given_up;
    if (gang_look(ws, at, tag, w)) return w;
    ++spins;
    if (spins > spin_limit) {
      gang_post(ws, abandon, 1.0f, tag);
      *gave_up = 1;
      return w;
    }
    if ((spins & 255) == 0 && gang_look(ws, abandon, tag, given_up)) {
      *gave_up = 1;
      return w;
    }
    __builtin_amdgcn_s_sleep(8);
  }
}

// which sums at tau = 1 a kernel keeps, see kd_gang_kernel
enum { kL1None = 0, kL1Own = 1, kL1Square = 2 };

// which of them a call runs
inline int l1_mode(const KdArgs& a) {
  if (!a.need_lse1) return kL1None;
  return 2.0f * a.c == kLog2e ? kL1Square : kL1Own;  // tau = 2 (halving a float is exact)
}

// words of scratch per slice: 3 per partial log-sum-exp, rounded up to a power of two
__host__ __device__ constexpr int gang_words(int ns) { return ns == 2 ? 8 : 16; }

// Zero-fills the share of slice `slice` of a gradient row's nvec groups: what a workgroup does when its row is not scored.
// Pieces of TH groups are dealt to the G workgroups in turn (`shift`: groups the pieces begin in front of the row), so that
// those that run side by side write side by side: (MI355X, rows that are not scored alone, TB/s, a run of up to 2,560 groups to
// each workgroup / this) 151,936 logits 5.35 / 5.9, 32,000 5.38 / 5.5, 50,003 4.83 / 5.3.
template <int K, int TH>
__device__ __forceinline__ void gang_zero_slice(uint16_t* grow, int nvec, int shift, int slice, int G, int tid) {
  const u32x4 z = {0, 0, 0, 0};
  u32x4* p = reinterpret_cast<u32x4*>(grow);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = (k * G + slice) * TH - shift + tid;
    if (i >= 0 && i < nvec) __builtin_nontemporal_store(z, p + i);
  }
}

// The same kernels with a row to a workgroup (SOLO: no exchange, no workspace) take rows that fit one: TH threads of K
// groups.  One wave per row (TH = 64) needs no barrier either; four such rows share a workgroup, which costs a quarter
// of the workgroups to start.
__host__ __device__ constexpr int solo_rows(int th) { return th == kWave ? 4 : 1; }
__host__ __device__ constexpr int gang_block(int th, bool solo) { return solo ? th * solo_rows(th) : th; }
// row of this workgroup (of this wave, where several rows share a workgroup)
template <int TH>
__device__ __forceinline__ int64_t solo_row() {
  if constexpr (solo_rows(TH) == 1) return blockIdx.x;
  return (int64_t)blockIdx.x * solo_rows(TH) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
}
// Groups per thread whose two fp32 values per pair of logits the skew forms keep in registers: the first two of a shared row's
// slice of seven are in LDS (16 KB each, four workgroups to a compute unit).  What these calls wait for is two exchanges per
// slice, and longer slices are fewer of them.  Measured (MI355X, 8,192 x 151,936, us, six groups in registers / five and two
// in LDS): skew KL 1234 / 1153, skew reverse KL 1264 / 1181, with a CE term at tau = 2 1342 / 1273; six in registers of seven
// or eight spill (1,423, 1,342); three workgroups of ten or eleven groups 1,169, 1,166; five groups 1,290, four with a fifth
// workgroup 1,353.
__host__ __device__ constexpr int skew_in_registers(int k, bool solo) { return !solo && k == 7 ? 5 : k; }
// waves per SIMD a kernel is compiled for: what its registers of data leave room for
__host__ __device__ constexpr int gang_waves(int data_registers) { return data_registers <= 32 ? 6 : 4; }
// orders a wave's or workgroup's earlier LDS accesses before its later ones
template <int TH>
__device__ __forceinline__ void row_sync() {
  if constexpr (TH == kWave)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  else
    __syncthreads();
}

// ---- the skew divergences (three sweeps): sums and gradient on normalised log2-probabilities.
//   skew KL          D = KL(p_T || m),  m = alpha p_T + (1 - alpha) p_S,  u = (alpha - 1) p_T / m
//   skew reverse KL  D = KL(p_S || m),  m = (1 - alpha) p_T + alpha p_S,  u = ln(p_S / m) + 1 - alpha p_S / m
// gradient = grad_scale / tau * p_S (u - ubar) with ubar = sum p_S u (+ ce_grad_scale p_S from the CE term at tau = 1).
// Entries of probability 0 (logits of -inf, underflow) contribute nothing: m has a floor, log ratios are kept finite.
struct SkewCoef {
  float c, Rs, Rt, izs, izt;  // p = 2^(x c - R) / z with the row's merged reference and sum (the reference is not
                              // folded into one logarithm: at logits in the thousands that would cost 2e-4 of p)
  float alpha, beta;          // beta = 1 - alpha
  float Av, B;                // gradient = Av v + B p_S, see skew_terms
  float C;                    // + C p_S^2: the CE term at tau = 2
};
constexpr float kSkewTiny = 1.0e-37f;

// Sweep 2 of an element, whose gradient is then finished from two fp32 values, p = p_S and v (g = grad_scale / tau,
// ce = ce_grad_scale):
//   skew KL          v = p_S p_T / m,                                       gradient = (alpha - 1) g v + (ce - g ubar) p
//   skew reverse KL  v = p_S (ln(p_S / m) - alpha p_S / m) = p_S (u - 1),   gradient = g v + (g (1 - ubar) + ce) p
// dsum: D in log2 units; usum = sum v.
template <int DIVK>
__device__ __forceinline__ void skew_terms(float ps, float pt, const SkewCoef& k, float& dsum, float& usum, float& p,
                                           float& v) {
  p = ps;
  // The floors are additive here (one fused operation each instead of a maximum): kSkewTiny changes nothing above
  // 2e-30, and below that the element's terms are far under one rounding step of the sums.  The log ratio is taken of
  // the quotient itself, which sweep 2 needs anyway.
  if constexpr (DIVK == kSkewKl) {
    const float m = __builtin_fmaf(k.alpha, pt, __builtin_fmaf(k.beta, ps, kSkewTiny));
    const float w = __builtin_fmaf(pt, __builtin_amdgcn_rcpf(m), kSkewTiny);  // p_T / m
    dsum = __builtin_fmaf(pt, __log2f(w), dsum);
    v = ps * w;
  } else {
    const float m = __builtin_fmaf(k.beta, pt, __builtin_fmaf(k.alpha, ps, kSkewTiny));
    const float t = __builtin_fmaf(ps, __builtin_amdgcn_rcpf(m), kSkewTiny);  // p_S / m
    const float l = __log2f(t);
    dsum = __builtin_fmaf(ps, l, dsum);
    v = ps * __builtin_fmaf(l, kLn2, t * -k.alpha);
  }
  usum += v;
}
// the same from logits (elements outside the cached slice: the sub-group tail of a row)
template <int DIVK>
__device__ __forceinline__ void skew_cache(float xs, float xt, const SkewCoef& k, float& dsum, float& usum, float& p,
                                           float& v) {
  skew_terms<DIVK>(exp2_fast(__builtin_fmaf(xs, k.c, -k.Rs)) * k.izs, exp2_fast(__builtin_fmaf(xt, k.c, -k.Rt)) * k.izt, k, dsum,
                   usum, p, v);
}
template <int DIVK>
__device__ __forceinline__ float skew_grad(float xs, float xt, const SkewCoef& k) {
  float d = 0.0f, u = 0.0f, p, v;
  skew_cache<DIVK>(xs, xt, k, d, u, p, v);
  return __builtin_fmaf(v, k.Av, k.B * p);
}

// K: groups per thread and tensor a workgroup holds.  A slice that is one run has at most a.gang_groups + shift <= K * 256 groups;
// dealt pieces cover the nvec + shift <= G * K * 256 groups from the boundary that the first one begins on (shift: 0 where all
// rows begin on 128-byte boundaries, else up to 7 groups, for which every slice is sized to 8 groups less).
// L1: what is summed at tau = 1 beside the sums at tau -- 0 nothing (tau = 1, or no such output wanted), kL1Own with
// exponentials of their own, kL1Square (tau = 2) from squares of the exponentials at tau.  Measured (MI355X, 4,096 x
// 151,936, dense teacher, composite loss at tau = 2): one workgroup per row, both sweeps from memory 738 us; shared
// rows with own exponentials 495 us, bound by the seven v_exp_f32 per pair of logits; squares, four of them, 462 us.
template <int K, int TEACHER, int L1, int DIVK = kForwardKl, int TH = kGangThreads, bool SOLO = false, bool GRAD = true>
__global__ __launch_bounds__(gang_block(TH, SOLO),
                             gang_waves(DIVK == kSkewKl || DIVK == kSkewReverseKl ? 16 * K : 8 * K)) void
kd_gang_kernel(const KdArgs a) {
  static_assert(TEACHER == kDense, "dense teacher");
  static_assert(SOLO || (TH == kGangThreads && GRAD), "shared rows: gradient calls, 256 threads");
  constexpr int GB = TH * 16;
  constexpr bool LSE1 = L1 != kL1None;
  constexpr int NS = LSE1 ? 4 : 2;  // 0 student / tau, 1 teacher / tau (+ cross), 2 student tau = 1, 3 teacher tau = 1
  constexpr int NW3 = NS * 3;
  constexpr int W = gang_words(NS);
  constexpr bool REV = DIVK == kReverseKl;
  // the skew forms take three sweeps over the registers and a second exchange: normalisers; D and ubar; gradient
  constexpr bool SKEW = DIVK == kSkewKl || DIVK == kSkewReverseKl;
  static_assert(NW3 + 2 <= W, "the second exchange of the skew forms uses two spare words of a slice's record");
  __shared__ float red[4 * 3 * (TH / kWave)];
  __shared__ uint32_t xch[SOLO ? 1 : kGangMax * W];
  __shared__ uint32_t xch2[SKEW && !SOLO ? kGangMax * 2 : 1];
  __shared__ int gave_up;
  constexpr int KR = skew_in_registers(K, SOLO), KL = SKEW ? K - KR : 0;  // groups [0, KL) of the skew forms' cache: LDS
  __shared__ float4 more[KL > 0 ? KL * 4 * TH : 1];

  const int G = SOLO ? 1 : a.gang;
  const int64_t row = SOLO ? solo_row<TH>() : (int64_t)(blockIdx.x / (unsigned)G);
  const int slice = SOLO ? 0 : (int)(blockIdx.x - (unsigned)(row * G));
  const int tid = threadIdx.x % (unsigned)TH;
  if constexpr (solo_rows(TH) > 1)
    if (row >= a.T) return;
  const int V = a.V;
  uint16_t* grow = GRAD ? a.g + row * a.s_stride : nullptr;
  const RowSplit sp = row_split(a.s + row * a.s_stride, V, true);  // all dense rows at one offset from a 16-byte boundary
  const int head = sp.head, nvec = sp.nvec, n_edge = V - nvec * 8;
  // The row's groups are dealt to its workgroups in pieces of TH groups (4 KB): piece k of slice `slice` is piece k G + slice of
  // the row.  Pieces begin on 128-byte boundaries of the gradient row's address (the first one is up to 7 groups shorter for
  // it), so that no cache line is shared by two workgroups.  A row's workgroups come out of the exchange together and write
  // side by side so.  Measured (MI355X, us, every workgroup one run of groups / this, both with the late label below):
  // 4,096 x 151,936 at tau = 2 with a CE term 446.9 / 435.6, 8,192 x 50,003 358.5 / 350.0, 16,384 x 32,000 reverse KL 458 / 451,
  // 6,001 x 65,536 355.8 / 348.2, 32,768 x 151,936 3,827 / 3,807; with all rows scored 32,000 506 / 495, 151,936 the same.
  // The skew forms with exponentials of their own at tau = 1, whose registers are full, take one run of gang_groups (up to 7
  // more) with the same boundaries (4,096 x 65,536 at tau = 3 with a CE term: 301, in pieces 315).
  // Group idx0 + k * step is the thread's k-th, if it is below `end`.  The last slice also owns the edge elements of the row.
  constexpr bool DEALT = !SOLO && !(SKEW && L1 == kL1Own);
  const bool last = SOLO || slice == G - 1;
  const int shift = SOLO ? 0 : (int)((reinterpret_cast<uintptr_t>(grow + head) >> 4) & 7u);
  const int run = slice * a.gang_groups - shift;
  const int first = DEALT ? slice * TH - shift : SOLO || slice == 0 ? 0 : (run < nvec ? run : nvec);
  const int step = DEALT ? G * TH : TH;
  const int end = DEALT || last ? nvec : (run + a.gang_groups < nvec ? run + a.gang_groups : nvec);
  const int idx0 = first + tid;  // < 0: in front of the row (k = 0 of slice 0)
  auto mine = [&](int k) __attribute__((always_inline)) { return idx0 < end - k * step && (!DEALT || k > 0 || idx0 >= 0); };

  if (!a.mask[row]) {  // not scored: scalars 0, the slice of the gradient row zero-filled, logits never read
    if (slice == 0 && tid == 0) {
      if (a.kd) a.kd[row] = 0.0f;
      if (a.nll) a.nll[row] = 0.0f;
      if (a.tnll) a.tnll[row] = 0.0f;
      if (a.lse) a.lse[row] = 0.0f;
    }
    if constexpr (GRAD) {
      gang_zero_slice<K, TH>(grow + head, nvec, shift, slice, G, tid);
      if (last && tid < n_edge) grow[sp.edge_elem(tid)] = 0;
    }
    return;
  }

  const uint16_t* srow = a.s + row * a.s_stride;
  const uint16_t* trow = a.t + row * a.t_stride;
  const float c = a.c;
  const bool lse1_t = LSE1 && a.tnll != nullptr;
  if (!SOLO && tid == 0) gave_up = 0;  // ordered before its use by the barrier of the workgroup's merge

  // The row as a buffer: all of a thread's groups are requested at once, unconditionally (a predicate around a load
  // makes the compiler wait for it on the spot); groups that are not the row's read as zero and are never used.
  const __amdgpu_buffer_rsrc_t rs = row_rsrc(srow + head, end);
  const __amdgpu_buffer_rsrc_t rt = row_rsrc(trow + head, end);
  const int voff = idx0 * 16;
  auto load = [&](const __amdgpu_buffer_rsrc_t& r, int k) __attribute__((always_inline)) {
    return !DEALT ? ld_group<GB>(r, voff, k, true, true) : ld_group<0>(r, voff + k * step * 16, 0, true, true);
  };
  uint4 sreg[K], treg[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    sreg[k] = load(rs, k);
    treg[k] = load(rt, k);
  }

  // The label logits belong to the slice that holds them (it reads them before it can overwrite them in place).  They arrive
  // behind the slice's groups, so that converting them at once would wait for all of those before the first is summed
  // (64 x 151,936 18.1 / 17.8 us, 32 x 32,000 12.6 / 12.3, 4,096 x 151,936 at tau = 2 451.6 / 446.9 us so, in a graph).
  int y = -1, k_own = -1, thread_y = 0;  // piece and thread of the label's group; -1: an edge element
  bool own_y = false;
  uint32_t s_y_bits = 0, t_y_bits = 0;
  if (a.labels) {
    y = a.labels[row];
    if ((unsigned)y < (unsigned)V) {
      const int gy = sp.group_of(y);
      if (gy >= 0) {
        const unsigned at = (unsigned)(gy + (DEALT ? shift : -first)), piece = at / TH;
        k_own = (int)(DEALT ? piece / (unsigned)G : piece);
        thread_y = (int)(at % TH);
        own_y = DEALT ? (int)(piece - (unsigned)(k_own * G)) == slice : gy >= first && gy < end;
      } else {
        own_y = last;
      }
      if (own_y) {
        s_y_bits = srow[y];
        t_y_bits = trow[y];
        if constexpr (SKEW) asm volatile("" : "+v"(s_y_bits), "+v"(t_y_bits));  // (their registers are full: waited for here)
      }
    }
  }
  const bool bad_label = a.labels && (unsigned)y >= (unsigned)V;  // uniform
  // The edge elements of the row, with the last slice: a latency more behind its sums if they are read there (64 x 50,003 15.4 /
  // 15.2 us; skew forms do, their registers are full)
  uint32_t s_e_bits = 0, t_e_bits = 0;
  auto read_edges = [&]() __attribute__((always_inline)) {
    const int e = sp.edge_elem(tid);
    s_e_bits = srow[e];
    t_e_bits = trow[e];
  };
  if (!SKEW && last && tid < n_edge) read_edges();

  Lse acc[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) acc[i].init();
  __builtin_amdgcn_sched_barrier(0);

  // ---- sweep 1 over the slice.  Fast form: a thread's reference exponents are fixed by its first group -- the
  // largest of its eight logits (integer maxima on the packed bit patterns, see pk_max_i16) plus kRefBias bits of
  // head room -- before the other groups have arrived, and no element is inspected again.  Terms are then 2^-100 and
  // below, sums stay far inside the fp32 range while no later logit exceeds the first group's by 2^200 (139 nats at
  // tau = 1), and a term that matters (within 2^-24 of the row's largest) cannot underflow.  What this form cannot take
  // -- a wider excursion, a logit of -inf (a masked vocabulary entry: 0 * -inf in the cross term) -- shows in the sums;
  // a wave that sees such a sum takes the careful form below (references that follow the data, guarded differences)
  // over the same registers.
  // The skew forms keep the exponentials of sweep 1 (two fp32 values per element pair, in place of the packed logits,
  // which are dead from here on -- hence the smaller K of these instances): sweep 2 scales them to probabilities with
  // one multiplication each instead of unpacking and exponentiating again, and leaves p_S and p_S (u - const) in the
  // same registers, so that the gradient sweep is one multiply-add per element.  Their references get 64 bits of head
  // room: an element's exponential is kept down to 2^-62 of the thread's first group's largest.
  // Rows of one workgroup, rows at any offset and calls with a CE term at tau != 1 take the largest of all the thread's
  // logits (thread_max) and no head room: arguments are then <= 0 to rounding and as small as can be where a term matters (rounding errors no larger than
  // in the streaming kernels that such rows once ran in, also on heavy tails and on rows of log-probabilities, and no
  // careful re-runs there), for half an instruction per logit and a wait for all loads, which short rows hide behind one
  // another.  (Measured on 4,096 x 151,936 with a CE term: tau = 2 650 us with the first group's reference, 655 with this
  // one; tau = 0.5 730 / 758, error of kd 2.1e-6 / 3.6e-7.)
  // Squares of exponentials get 44 bits, so that a square is kept down to 2^-38 of the first group's largest square and
  // its sum is inside the range up to 94 bits above the first group's largest logit.
  const bool ref_of_all = SOLO || a.ragged || (LSE1 && a.cscale != 0.0f);  // uniform
  const float kRefBias = ref_of_all ? 0.0f : (L1 == kL1Square ? 44.0f : (SKEW ? 64.0f : 100.0f));
  float cp[SKEW ? KR : 1][8], cv[SKEW ? KR : 1][8];
  auto cache_get = [&](int k, float (&p)[8], float (&v)[8]) __attribute__((always_inline)) {
    if (k >= KL) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        p[j] = cp[k - KL][j];
        v[j] = cv[k - KL][j];
      }
    } else {  // (a thread reads its own words only: no barrier)
      const float4* m = more + k * 4 * TH + tid;
      const float4 w[4] = {m[0], m[TH], m[2 * TH], m[3 * TH]};
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        p[4 * j] = w[j].x; p[4 * j + 1] = w[j].y; p[4 * j + 2] = w[j].z; p[4 * j + 3] = w[j].w;
        v[4 * j] = w[2 + j].x; v[4 * j + 1] = w[2 + j].y; v[4 * j + 2] = w[2 + j].z; v[4 * j + 3] = w[2 + j].w;
      }
    }
  };
  auto cache_put = [&](int k, const float (&p)[8], const float (&v)[8]) __attribute__((always_inline)) {
    if (k >= KL) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        cp[k - KL][j] = p[j];
        cv[k - KL][j] = v[j];
      }
    } else {
      float4* m = more + k * 4 * TH + tid;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        m[j * TH] = make_float4(p[4 * j], p[4 * j + 1], p[4 * j + 2], p[4 * j + 3]);
        m[(2 + j) * TH] = make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
      }
    }
  };
  if (mine(0) || (DEALT && mine(1))) {  // (threads without a group keep their empty partials)
    float fs, ft;
    if (ref_of_all) {
      fs = thread_max<DEALT>(sreg, mine);
      ft = thread_max<DEALT>(treg, mine);
    } else {
      uint32_t ms = pk_max_group(sreg[0]), mt = pk_max_group(treg[0]);
      if (DEALT && idx0 < 0) {
        ms = pk_max_group(sreg[1]);
        mt = pk_max_group(treg[1]);
      }
      fs = pk_max_value(ms);
      ft = pk_max_value(mt);
    }
    acc[0].r = __builtin_rintf(__builtin_fmaxf(__builtin_fmaf(fs, c, kRefBias), -1.0e30f));
    acc[1].r = __builtin_rintf(__builtin_fmaxf(__builtin_fmaf(ft, c, kRefBias), -1.0e30f));
    if constexpr (L1 == kL1Own) {
      acc[2].r = __builtin_rintf(__builtin_fmaxf(__builtin_fmaf(fs, kLog2e, kRefBias), -1.0e30f));
      acc[3].r = __builtin_rintf(__builtin_fmaxf(__builtin_fmaf(ft, kLog2e, kRefBias), -1.0e30f));
    }
    if constexpr (L1 == kL1Square) {
      acc[2].r = 2.0f * acc[0].r;
      acc[3].r = 2.0f * acc[1].r;
    }
  }
  // The forward and the reverse KL unpack with the matrix cores (a logit that is not finite shows in the sums as above) where
  // a thread has more than four groups; shorter rows wait for latencies, not for the vector ALUs.  Measured (MI355X, us,
  // shifts and masks / this, same bits; with the shorter merges and the folded form without its sign): 8,192 rows of 50,003
  // 376 / 364, 24,576 at tau = 2 232 / 210 and with a CE term 251 / 221, 50,304 at tau = 2 424 / 400, 4,096 x 151,936 at
  // tau = 2 with a CE term 458 / 453; 64 rows of 4,096 (four groups per thread) 4.9 / 5.2.
  constexpr bool MFMA = !SKEW && K > 4;
  const s16x4 identity = lane_identity(kBf16One);
  const int wave0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
  auto add_group = [&](const float (&xs)[8], const float (&xt)[8], const float (&d)[8], int k) __attribute__((always_inline)) {
    float p[8], v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float es = exp2_fast(__builtin_fmaf(xs[j], c, -acc[0].r));
      const float et = exp2_fast(__builtin_fmaf(xt[j], c, -acc[1].r));
      acc[0].z += es;
      acc[1].z += et;
      if constexpr (REV)
        acc[0].a = __builtin_fmaf(es, MFMA ? d[j] : xs[j] - xt[j], acc[0].a);
      else if constexpr (!SKEW)
        acc[1].a = __builtin_fmaf(et, MFMA ? d[j] : xt[j] - xs[j], acc[1].a);
      p[j] = es;
      v[j] = et;
      if constexpr (L1 == kL1Square) {
        acc[2].z = __builtin_fmaf(es, es, acc[2].z);
        acc[3].z = __builtin_fmaf(et, et, acc[3].z);
      }
      if constexpr (L1 == kL1Own) {
        acc[2].z += exp2_fast(__builtin_fmaf(xs[j], kLog2e, -acc[2].r));
        if (lse1_t) acc[3].z += exp2_fast(__builtin_fmaf(xt[j], kLog2e, -acc[3].r));
      }
    }
    if constexpr (SKEW) cache_put(k, p, v);
  };
#pragma unroll
  for (int k = 0; k < K; ++k) {
    float xs[8], xt[8], d[8] = {};
    if constexpr (MFMA) {
      if (first + wave0 < end - k * step) {  // uniform: a group for the wave's first lane at least
        unpack8_mfma(sreg[k], identity, xs);
        unpack8_mfma(treg[k], identity, xt);
        const s16x4 minus = identity ^ (short)0x8000;
        if constexpr (REV)
          mfma8(treg[k], minus, xs, d);
        else
          mfma8(sreg[k], minus, xt, d);
        if (mine(k)) add_group(xs, xt, d, k);
      }
    } else if (mine(k)) {
      unpack8(sreg[k], xs);
      unpack8(treg[k], xt);
      add_group(xs, xt, d, k);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  bool all_finite = true;  // wave-uniform: no infinity or NaN among the wave's logits
  {
    constexpr float kBig = 1.2676506e30f;  // 2^100
    bool odd = false;
#pragma unroll
    for (int i = 0; i < NS; ++i) odd = odd || !(acc[i].z < kBig) || !(fabsf(acc[i].a) < kBig);
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {  // wave-uniform
      all_finite = false;
#pragma unroll
      for (int i = 0; i < NS; ++i) acc[i].init();
      if constexpr (SKEW) {  // the packed logits are gone: fetched again (rare; they are still in a cache)
#pragma unroll
        for (int k = 0; k < K; ++k) {
          sreg[k] = load(rs, k);
          treg[k] = load(rt, k);
        }
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (mine(k)) accum8<kDense, LSE1, REV>(sreg[k], treg[k], c, lse1_t, acc);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (SKEW) {  // the exponentials again, against the references the careful form ended with
#pragma unroll
        for (int k = 0; k < K; ++k) {  // (every group, also those past the slice's end: all of the cache is rewritten)
          float xs[8], xt[8], p[8], v[8];
          unpack8(sreg[k], xs);
          unpack8(treg[k], xt);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            p[j] = exp2_fast(__builtin_fmaf(xs[j], c, -acc[0].r));
            v[j] = exp2_fast(__builtin_fmaf(xt[j], c, -acc[1].r));
          }
          cache_put(k, p, v);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
  const float r_s_thread = acc[0].r, r_t_thread = acc[1].r;  // what this thread's cached exponentials refer to
  // the conversions stay here: behind the sums, and in front of this workgroup's post (rows in place)
  if constexpr (!SKEW) asm volatile("" : "+v"(s_y_bits), "+v"(t_y_bits), "+v"(s_e_bits), "+v"(t_e_bits));
  if (last && tid < n_edge) {
    if constexpr (SKEW) read_edges();
    const float xs = bf16_lo(s_e_bits), xt = bf16_lo(t_e_bits);
    if constexpr (REV) {
      acc[1].add1(xt, c);
      acc[0].add1_cross(xs, xs - xt, c);
    } else {
      acc[1].add1_cross(xt, xt - xs, c);
      acc[0].add1(xs, c);
    }
    if constexpr (LSE1) {
      if (lse1_t) acc[3].add1(xt, kLog2e);
      acc[2].add1(xs, kLog2e);
    }
  }

  // ---- wave totals, workgroup totals (through LDS), post, wait for the row's, row totals: the same merge each time
  const int lane = tid & (kWave - 1), wid = tid / kWave;
  constexpr int NWV = TH / kWave;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    normalise(acc[i]);
    if (i == (REV ? 0 : 1) && !SKEW)  // the stream that carries the cross term
      wave_merge_rescaled<true>(acc[i]);
    else
      wave_merge_rescaled<false>(acc[i]);
  }
  bool timeout = false;
  const size_t rec = SOLO ? 0 : (size_t)blockIdx.x * W;      // words of scratch[row][slice]
  const size_t abandon = SOLO ? 0 : (size_t)gridDim.x * W;  // behind the record
  if constexpr (NWV > 1) {
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        red[(i * 3 + 0) * NWV + wid] = acc[i].r;
        red[(i * 3 + 1) * NWV + wid] = acc[i].z;
        red[(i * 3 + 2) * NWV + wid] = acc[i].a;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      acc[i].init();
      if (lane < NWV) {
        acc[i].r = red[(i * 3 + 0) * NWV + lane];
        acc[i].z = red[(i * 3 + 1) * NWV + lane];
        acc[i].a = red[(i * 3 + 2) * NWV + lane];
      }
      if (i == (REV ? 0 : 1) && !SKEW)  // the stream that carries the cross term
        wave_merge_rescaled<true, merge_lanes(NWV)>(acc[i]);
      else
        wave_merge_rescaled<false, merge_lanes(NWV)>(acc[i]);
    }

  }
  if constexpr (!SOLO) {
    if (tid < NW3) {
      float v = acc[0].r;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        if (tid == i * 3 + 0) v = acc[i].r;
        if (tid == i * 3 + 1) v = acc[i].z;
        if (tid == i * 3 + 2) v = acc[i].a;
      }
      gang_post(a.ws, rec + tid, v, a.tag);
    }
    {
      const size_t rrow = (size_t)row * G * W;
      const int nw = G * NW3;
      for (int w = tid; w < nw; w += TH) {
        const int s = w / NW3, f = w - s * NW3;
        xch[s * W + f] = gang_wait(a.ws, rrow + s * W + f, abandon, a.tag, a.spin_limit, &gave_up);
      }
    }
    __syncthreads();
    timeout = gave_up != 0;  // uniform
#pragma unroll
    for (int i = 0; i < NS; ++i) {  // lane s < G takes slice s: every wave of every workgroup of the row computes the
      acc[i].init();                // same totals in the same order
      if (lane < G) {
        acc[i].r = __builtin_bit_cast(float, xch[lane * W + i * 3 + 0]);
        acc[i].z = __builtin_bit_cast(float, xch[lane * W + i * 3 + 1]);
        acc[i].a = __builtin_bit_cast(float, xch[lane * W + i * 3 + 2]);
      }
      constexpr bool kCross = !SKEW;
      if (G <= 16) {  // uniform
        if (kCross && i == (REV ? 0 : 1))  // the stream that carries the cross term
          wave_merge_rescaled<true, 16>(acc[i]);
        else
          wave_merge_rescaled<false, 16>(acc[i]);
      } else {
        if (kCross && i == (REV ? 0 : 1))
          wave_merge_rescaled<true>(acc[i]);
        else
          wave_merge_rescaled<false>(acc[i]);
      }
    }
  }

  const float s_y = bf16_lo(s_y_bits), t_y = bf16_lo(t_y_bits);
  const float Ls = acc[0].log2_sum();
  const float Lt = acc[1].log2_sum();
  const float lse1_s = __fmul_rn(LSE1 ? acc[NS - 2].log2_sum() : Ls, kLn2);
  const float lse_diff = ((acc[0].r - acc[1].r) + (acc[0].log2_z() - acc[1].log2_z())) * kLn2;  // lse_S - lse_T at tau
  float kd = REV ? (acc[0].a / acc[0].z) * a.inv_tau - lse_diff : (acc[1].a / acc[1].z) * a.inv_tau + lse_diff;
  kd = kd < 0.0f ? 0.0f : kd;  // (the skew forms replace it below)
  // uniform.  With a CE term at tau != 1 (LSE1) the gradient takes a third exponential per element, against the
  // student's normaliser at tau = 1 that sweep 1 has summed anyway.
  const bool ce = a.cscale != 0.0f;
  const float cs_shared = LSE1 ? 0.0f : a.cscale;  // weight of a CE term that shares the KD term's softmax
  Sweep2Coef kf = folded_coef(acc[0], acc[1], c, a.gscale, a.cscale, true, LSE1);
  kf.folded = kf.folded && !a.ragged && !(SOLO && V < kCachedMinVocab);
  if (!MFMA || REV || !kf.folded || last || (ce && own_y))  // uniform: the folded form alone needs none of these quotients
    set_precise_coef(kf, acc[0], acc[1], acc[LSE1 ? 2 : 0], c, a.gscale, a.cscale, true, LSE1);
  SkewCoef ks;
  if constexpr (SKEW) {
    // ---- sweep 2 of the skew forms over the registers: D and ubar need the row's normalisers in every term
    ks.c = c;
    ks.Rs = acc[0].r;
    ks.Rt = acc[1].r;
    ks.izs = 1.0f / acc[0].z;
    ks.izt = 1.0f / acc[1].z;
    ks.alpha = a.alpha;
    ks.beta = 1.0f - a.alpha;
    float dsum = 0.0f, usum = 0.0f;
    // cached exponential -> probability
    const float fs = exp2_fast(r_s_thread - ks.Rs) * ks.izs, ft = exp2_fast(r_t_thread - ks.Rt) * ks.izt;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (mine(k)) {
        float p[8], v[8];
        cache_get(k, p, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) skew_terms<DIVK>(p[j] * fs, v[j] * ft, ks, dsum, usum, p[j], v[j]);
        cache_put(k, p, v);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (last && tid < n_edge) {
      read_edges();
      float p, v;
      skew_cache<DIVK>(bf16_lo(s_e_bits), bf16_lo(t_e_bits), ks, dsum, usum, p, v);
    }
    // workgroup totals, second post / wait, row totals -- plain sums in a fixed order
    dsum = wave_sum_dpp(dsum);
    usum = wave_sum_dpp(usum);
    if constexpr (NWV > 1) {
      if constexpr (SOLO) __syncthreads();  // the first merge's readers of `red` are done
      if (lane == 0) {
        red[wid] = dsum;
        red[NWV + wid] = usum;
      }
      __syncthreads();
      dsum = wave_sum_dpp(lane < NWV ? red[lane] : 0.0f);
      usum = wave_sum_dpp(lane < NWV ? red[NWV + lane] : 0.0f);
    }
    if constexpr (!SOLO) {
      if (tid < 2) gang_post(a.ws, rec + NW3 + tid, tid == 0 ? dsum : usum, a.tag);
      {
        const size_t rrow = (size_t)row * G * W;
        for (int w = tid; w < 2 * G; w += TH) {
          const int s = w >> 1, f = w & 1;
          xch2[w] = gang_wait(a.ws, rrow + s * W + NW3 + f, abandon, a.tag, a.spin_limit, &gave_up);
        }
      }
      __syncthreads();
      timeout = gave_up != 0;
      dsum = wave_sum_dpp(lane < G ? __builtin_bit_cast(float, xch2[2 * lane]) : 0.0f);
      usum = wave_sum_dpp(lane < G ? __builtin_bit_cast(float, xch2[2 * lane + 1]) : 0.0f);
    }
    kd = dsum * kLn2;
    kd = kd < 0.0f ? 0.0f : kd;
    const float g = a.gscale;  // (grad_scale / tau)
    ks.C = kf.wc_square * acc[0].z * acc[0].z;  // Softmax(s) = e_S^2 / (...), e_S = p_S z_S
    if constexpr (DIVK == kSkewKl) {
      const float ubar = (a.alpha - 1.0f) * usum;
      ks.Av = (a.alpha - 1.0f) * g;
      ks.B = cs_shared - g * ubar;
    } else {
      const float ubar = usum + 1.0f;
      ks.B = __builtin_fmaf(g, 1.0f - ubar, cs_shared);
      ks.Av = g;
    }
  }
  if constexpr (REV) {
    const float inv_z = 1.0f / acc[0].z;
    kf.ra = a.gscale * a.inv_tau * inv_z;
    kf.rb = (cs_shared - a.gscale * (lse_diff + kd)) * inv_z;
    kf.folded = true;
  }

  if (tid == 0) {
    const float nanv = __builtin_nanf("");
    int flags = 0;
    if (slice == 0) {
      if (timeout) flags |= 8;
      if (bad_label && (a.nll || a.tnll || ce)) flags |= 1;
      if (a.kd) a.kd[row] = timeout ? nanv : kd;
      if (a.lse) a.lse[row] = timeout ? nanv : lse1_s;
      if (bad_label) {
        if (a.nll) a.nll[row] = nanv;
        if (a.tnll) a.tnll[row] = nanv;
      }
    } else if (timeout) {
      flags |= 8;
    }
    if (own_y) {
      if (a.nll) a.nll[row] = timeout ? nanv : __fsub_rn(lse1_s, s_y);
      if (a.tnll) {
        const float lse1_tt = __fmul_rn(LSE1 ? acc[NS - 1].log2_sum() : Lt, kLn2);
        a.tnll[row] = timeout ? nanv : __fsub_rn(lse1_tt, t_y);
      }
    }
    if (flags && a.status) atomicOr(a.status, flags);
  }

  if constexpr (!GRAD) return;
  // ---- sweep 2: the gradient of the slice, from the registers, last group first
  uint8_t* gslice = reinterpret_cast<uint8_t*>(grow + head) + (int64_t)first * 16;
  auto store = [&](int k, const uint4& o) {  // the group's base is uniform, the thread adds tid * 16
    const u32x4 w = {o.x, o.y, o.z, o.w};
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(gslice + (size_t)k * (step * 16)) + tid);
  };
  if (timeout || (ce && bad_label)) {  // uniform: the row cannot be differentiated
    const uint4 qnan = make_uint4(0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (mine(k)) store(k, qnan);
    if (last && tid < n_edge) grow[sp.edge_elem(tid)] = 0x7fc0;
    return;
  }
  // The label position of the composite loss (Eq. 1) gets its final value from fp32, rounded once: the group that
  // holds it is the same for every thread (k_y, uniform), the thread that owns it keeps a mask and the bits.
  int k_y = -1;
  uint4 y_keep = make_uint4(~0u, ~0u, ~0u, ~0u), y_bits = make_uint4(0, 0, 0, 0);
  uint16_t y_tail = 0;
  if (ce && own_y) {  // uniform
    float gy;
    if constexpr (REV)
      gy = grad_reverse_elem(s_y, t_y, kf);
    else if constexpr (SKEW)
      gy = skew_grad<DIVK>(s_y, t_y, ks);
    else
      gy = grad_dense_elem(s_y, t_y, kf.p);
    if constexpr (LSE1 && (REV || SKEW)) gy = add_ce_own(gy, s_y, kf.p);
    const uint32_t b16 = one_bf16(gy - a.cscale);
    y_tail = (uint16_t)b16;
    if (k_own >= 0) {
      k_y = k_own;
      if (thread_y == tid) {
        const int j = (y - head) & 7;
        const uint32_t keep = (j & 1) ? 0x0000ffffu : 0xffff0000u, bits = (j & 1) ? b16 << 16 : b16;
        if ((j >> 1) == 0) { y_keep.x = keep; y_bits.x = bits; }
        if ((j >> 1) == 1) { y_keep.y = keep; y_bits.y = bits; }
        if ((j >> 1) == 2) { y_keep.z = keep; y_bits.z = bits; }
        if ((j >> 1) == 3) { y_keep.w = keep; y_bits.w = bits; }
      }
    }
  }
  auto patch_label = [&](uint4& o) {  // a no-op in every thread but the one that owns the label
    o.x = (o.x & y_keep.x) | y_bits.x;
    o.y = (o.y & y_keep.y) | y_bits.y;
    o.z = (o.z & y_keep.z) | y_bits.z;
    o.w = (o.w & y_keep.w) | y_bits.w;
  };
  if (last && tid < n_edge) {
    const int e = sp.edge_elem(tid);
    if constexpr (SKEW) read_edges();
    const float xs = bf16_lo(s_e_bits), xt = bf16_lo(t_e_bits);
    float ge;
    if constexpr (SKEW)
      ge = skew_grad<DIVK>(xs, xt, ks);
    else
      ge = REV ? grad_reverse_elem(xs, xt, kf) : grad_dense_elem(xs, xt, kf.p);
    if constexpr (LSE1 && (REV || SKEW))
      if (ce) ge = add_ce_own(ge, xs, kf.p);
    uint16_t o = one_bf16(ge);
    if (ce && own_y && e == y) o = y_tail;
    grow[e] = o;
  }
  // The walk over the slice, last group first.  Unpacked again from the packed registers (`opaque`) instead of keeping
  // sweep 1's floats alive.
  auto walk_unpacked = [&](auto form, auto mfma) __attribute__((always_inline)) {
    constexpr int FORM = decltype(form)::value;
    constexpr bool M = decltype(mfma)::value;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
      if constexpr (MFMA)
        if (first + wave0 >= end - k * step) continue;  // uniform
      opaque(sreg[k]);
      opaque(treg[k]);
      uint4 o = grad8<kDense, FORM, DIVK, M>(sreg[k], treg[k], kf, identity);
      if (k == k_y) patch_label(o);  // uniform
      if (mine(k)) store(k, o);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto walk = [&](auto form) __attribute__((always_inline)) {
    if constexpr (MFMA) {
      if (all_finite) {  // wave-uniform
        walk_unpacked(form, std::true_type{});
        return;
      }
    }
    walk_unpacked(form, std::false_type{});
  };
  if constexpr (SKEW) {
    if (L1 == kL1Own && ce) {  // uniform: the packed student logits are gone, their slice is fetched again (this workgroup has
                       // not overwritten it yet, and no other one does)
#pragma unroll
      for (int k = K - 1; k >= 0; --k) {
        const uint4 vs = load(rs, k);
        float xs[8], gv[8], p[8], v[8];
        unpack8(vs, xs);
        cache_get(k, p, v);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          gv[j] = add_ce_own(__builtin_fmaf(v[j], ks.Av, ks.B * p[j]), xs[j], kf.p);
        uint4 o = make_uint4(pack_bf16(gv[0], gv[1]), pack_bf16(gv[2], gv[3]), pack_bf16(gv[4], gv[5]), pack_bf16(gv[6], gv[7]));
        if (k == k_y) patch_label(o);  // uniform
        if (mine(k)) store(k, o);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int k = K - 1; k >= 0; --k) {
        float gv[8], p[8], v[8];
        cache_get(k, p, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if constexpr (L1 == kL1Square)  // (ks.C = 0 without a CE term)
            gv[j] = __builtin_fmaf(v[j], ks.Av, __builtin_fmaf(ks.C, p[j], ks.B) * p[j]);
          else
            gv[j] = __builtin_fmaf(v[j], ks.Av, ks.B * p[j]);
        }
        uint4 o = make_uint4(pack_bf16(gv[0], gv[1]), pack_bf16(gv[2], gv[3]), pack_bf16(gv[4], gv[5]), pack_bf16(gv[6], gv[7]));
        if (k == k_y) patch_label(o);  // uniform
        if (mine(k)) store(k, o);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else if (LSE1 && ce) {  // uniform
    walk(std::integral_constant<int, L1 == kL1Square ? kPreciseCeSquare : kPreciseCeOwn>{});
  } else if (MFMA && kf.folded && (REV || kf.sign == 0)) {  // uniform
    walk(std::integral_constant<int, kFoldedPlus>{});
  } else if (kf.folded) {
    walk(std::integral_constant<int, kFolded>{});
  } else if (ce) {  // rows at any offset, or whose reference exponents are in the thousands: precise form
    walk(std::integral_constant<int, kPreciseCe>{});
  } else {
    walk(std::integral_constant<int, kPrecise>{});
  }
}

}  // namespace npd
