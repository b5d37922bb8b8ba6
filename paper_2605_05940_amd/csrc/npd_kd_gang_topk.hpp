// Row-gang kernel for a top-k teacher (Sec. 3.1: the teacher is stored as k vocabulary ids + k values per position;
// Eq. 2 with p_T renormalised over the k stored entries and p_S over the full vocabulary).  Same scheme as
// npd_kd_gang.hpp -- a row shared by G short-lived workgroups of 256 threads, the student slice in registers, partial
// log-sum-exps exchanged through the scratch record -- with these differences:
//   - only the student row is dense: one read and one write per logit;
//   - every workgroup of a row reads the row's whole top-k record (k ids + k values, a few hundred bytes): the teacher's
//     normaliser over the k values is computed by each of them, the support positions that fall into its own slice get
//     their final values (from fp32, rounded once), and slice 0 also gathers the student logits of all k support
//     positions for kd_tok;
//   - every student logit a workgroup needs from outside its registers (support positions, the label) is fetched
//     before the workgroup posts its partial sum, i.e. before any workgroup of the row can overwrite the row in place.
#pragma once
#include "npd_kd_gang.hpp"

namespace npd {

// SOLO, TH, GRAD: as in npd_kd_gang.hpp; the forward-only SOLO form also takes calls without a teacher (k = 0).
// Dynamic LDS: topk_lds_words per row of the workgroup.
//
// The final values of the support positions are put into the groups before they are stored: each group of the workgroup has
// a list of them in LDS that the threads build with exchanges (its order does not matter: the ids are distinct).
// Stored behind the dense values they cost a wait for the whole workgroup's stores, the ids once more and k partial lines per
// row (MI355X, us, so / with lists: 65,536 rows of 4,096, k = 64, one workgroup each 412 / 255; shared rows, with the record
// requested in front of the slice's logits and its support logits gathered behind them, k = 64: 8,192 of 50,304 263 / 258,
// of 36,000 194 / 184, 4,096 of 65,536 159 / 152, 64 of 151,936 16.0 / 15.5; k = 250, 8,192 of 128,256 681 / 625;
// k = 1,000, 4,096 of 151,936 542 / 496).
constexpr int kMaxEdges = 16;
__host__ __device__ constexpr int topk_lds_words(int th, int groups, int k, bool lists) {
  return (lists ? th * groups + kMaxEdges + k : 0) + (k + 1) / 2;
}

template <int K, int L1, int TH = kGangThreads, bool SOLO = false, bool GRAD = true, bool DEALT = false>
__global__ __launch_bounds__(gang_block(TH, SOLO), SOLO && K <= 8 ? 8 : 6) void
kd_gang_topk_kernel(const KdArgs a) {
  static_assert(SOLO || (TH == kGangThreads && GRAD), "shared rows: gradient calls, 256 threads");
  static_assert(!SOLO || !DEALT, "one workgroup takes the whole row");
  constexpr int GB = TH * 16;
  constexpr bool LSE1 = L1 != kL1None;
  constexpr int NS = LSE1 ? 2 : 1;  // student / tau, student at tau = 1
  constexpr int NW3 = NS * 3;
  constexpr int W = 8;              // words of scratch per slice
  constexpr int NWV = TH / kWave;
  __shared__ float red[2 * 3 * NWV + NWV];
  __shared__ uint32_t xch[SOLO ? 1 : kGangMax * W];
  extern __shared__ uint32_t topk_rows[];
  __shared__ int gave_up, y_hit_row;

  const int G = SOLO ? 1 : a.gang;
  const int64_t row = SOLO ? solo_row<TH>() : (int64_t)(blockIdx.x / (unsigned)G);
  const int slice = SOLO ? 0 : (int)(blockIdx.x - (unsigned)(row * G));
  const int tid = threadIdx.x % (unsigned)TH;
  if constexpr (solo_rows(TH) > 1)
    if (row >= a.T) return;
  const int k_top = a.k;
  // LDS of the row: per group (and per edge element) the first of its support positions (entry + 1, 0: none), per entry
  // the next one of the same group (same encoding, low half) and its element of the group (high half); the student
  // logits at the support positions (bf16 bits), later their final gradient values
  uint32_t* first = topk_rows + (solo_rows(TH) > 1 ? (threadIdx.x / TH) * topk_lds_words(TH, K, k_top, GRAD) : 0);
  uint32_t* link = first + K * TH + kMaxEdges;
  uint16_t* sup_s = reinterpret_cast<uint16_t*>(GRAD ? link + k_top : first);
  if constexpr (GRAD) {  // ordered before their use by the barrier below
#pragma unroll
    for (int k = 0; k < K; ++k) first[k * TH + tid] = 0;
    if (tid < kMaxEdges) first[K * TH + tid] = 0;
  }
  const int V = a.V;
  uint16_t* grow = GRAD ? a.g + row * a.s_stride : nullptr;
  const RowSplit sp = row_split(a.s + row * a.s_stride, V, true);  // all dense rows at one offset from a 16-byte boundary
  const int head = sp.head, nvec = sp.nvec, n_edge = V - nvec * 8;
  // Slices: one run of gang_groups (up to 7 more), or, DEALT (rows that begin inside a 16-byte group), pieces of TH groups dealt to
  // the row's workgroups in turn; boundaries as in npd_kd_gang.hpp.  Measured (MI355X, us, k = 64, runs / pieces): 8,192 x 50,003
  // 268 / 261; aligned rows of 151,936 at tau = 2 726 / 733, 4,096 of 262,144 567 / 569, of 65,536 152 / 151.  Group
  // idx0 + k * step is the thread's k-th, if it is below `end`.  The last slice also owns the edge elements of the row.
  const bool last = SOLO || slice == G - 1;
  const int shift = SOLO ? 0 : (int)((reinterpret_cast<uintptr_t>(grow + head) >> 4) & 7u);
  const int run = slice * a.gang_groups - shift;
  const int first_group = DEALT ? slice * TH - shift : SOLO || slice == 0 ? 0 : (run < nvec ? run : nvec);
  const int step = DEALT ? G * TH : TH;
  const int end = DEALT || last ? nvec : (run + a.gang_groups < nvec ? run + a.gang_groups : nvec);
  const int idx0 = first_group + tid;  // < 0: in front of the row (k = 0 of slice 0)
  auto mine = [&](int k) __attribute__((always_inline)) { return idx0 < end - k * step && (!DEALT || k > 0 || idx0 >= 0); };

  if (!a.mask[row]) {  // not scored: scalars 0, the slice of the gradient row zero-filled, logits never read
    if (slice == 0 && tid == 0) {
      if (a.kd) a.kd[row] = 0.0f;
      if (a.nll) a.nll[row] = 0.0f;
      if (a.lse) a.lse[row] = 0.0f;
    }
    if constexpr (GRAD) {
      gang_zero_slice<K, TH>(grow + head, nvec, shift, slice, G, tid);
      if (last && tid < n_edge) grow[sp.edge_elem(tid)] = 0;
    }
    return;
  }

  const uint16_t* srow = a.s + row * a.s_stride;
  const float c = a.c;
  if (TH > kWave && tid == 0) gave_up = y_hit_row = 0;  // ordered before their use by the barrier below

  // ---- the row's top-k record: entries tid, tid + TH, ...; the first (for k <= TH the only one) is kept in registers and
  // requested in front of the slice (what is loaded behind it arrives behind it)
  const int32_t* irow = a.tidx + row * (int64_t)k_top;
  const float* vrow = a.tval + row * (int64_t)k_top;
  const bool has_entry = tid < k_top;
  const int id_first = has_entry ? irow[tid] : 0;
  const float v_first = has_entry ? vrow[tid] : 0.0f;
  __builtin_amdgcn_sched_barrier(0);

  const __amdgpu_buffer_rsrc_t rs = row_rsrc(srow + head, end);
  const int voff = idx0 * 16;
  uint4 sreg[K];
#pragma unroll
  for (int k = 0; k < K; ++k)
    sreg[k] = !DEALT ? ld_group<GB>(rs, voff, k, true, true) : ld_group<0>(rs, voff + k * step * 16, 0, true, true);
  __builtin_amdgcn_sched_barrier(0);

  // place of element e among this workgroup's: k * TH + thread of its group, behind K * TH the edge elements (the last slice's);
  // -1: another workgroup's
  auto place = [&](int e) __attribute__((always_inline)) {
    const int ge = sp.group_of(e);
    if (ge < 0) return last ? K * TH + (e < head ? e : e - nvec * 8) : -1;
    if constexpr (SOLO) return ge;
    if constexpr (!DEALT) return ge >= first_group && ge < end ? ge - first_group : -1;
    const unsigned at = (unsigned)(ge + shift), piece = at / TH, k = piece / (unsigned)G;
    return (int)(piece - k * (unsigned)G) == slice ? (int)(k * TH + at % TH) : -1;
  };
  // student logits from outside the registers: the label's, and those at the support positions this workgroup will need
  // (its own; all of them in slice 0)
  int y = -1, place_y = -1;
  uint32_t s_y_bits = 0;
  if (a.labels) {
    y = a.labels[row];
    if ((unsigned)y < (unsigned)V) place_y = place(y);
    if (place_y >= 0) s_y_bits = srow[y];
  }
  const bool own_y = place_y >= 0;
  const bool bad_label = a.labels && (unsigned)y >= (unsigned)V;  // uniform
  auto needs = [&](int id) __attribute__((always_inline)) { return (unsigned)id < (unsigned)V && (slice == 0 || place(id) >= 0); };
  uint32_t sup_first = 0, s_e_bits = 0;
  if (has_entry && needs(id_first)) sup_first = srow[id_first];
  if (last && tid < n_edge) s_e_bits = srow[sp.edge_elem(tid)];

  // ---- sweep 1 over the student slice (see npd_kd_gang.hpp: fixed reference from the first group, careful re-run
  // of a wave whose sums show an anomaly)
  Lse acc[4];  // 0 student / tau, 2 student at tau = 1 (the indices accum8 uses; 1 and 3 stay empty)
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i].init();
  const bool ref_of_all = SOLO || a.ragged || (LSE1 && a.cscale != 0.0f);  // see npd_kd_gang.hpp
  const float kRefBias = ref_of_all ? 0.0f : (L1 == kL1Square ? 44.0f : 100.0f);  // see npd_kd_gang.hpp
  if (mine(0) || (DEALT && mine(1))) {
    uint32_t ms = pk_max_group(sreg[0]);
    if (DEALT && idx0 < 0) ms = pk_max_group(sreg[1]);
    const float fs = ref_of_all ? thread_max<DEALT>(sreg, mine) : pk_max_value(ms);
    acc[0].r = __builtin_rintf(__builtin_fmaxf(__builtin_fmaf(fs, c, kRefBias), -1.0e30f));
    if constexpr (L1 == kL1Own) acc[2].r = __builtin_rintf(__builtin_fmaxf(__builtin_fmaf(fs, kLog2e, kRefBias), -1.0e30f));
    if constexpr (L1 == kL1Square) acc[2].r = 2.0f * acc[0].r;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (mine(k)) {
      float xs[8];
      unpack8(sreg[k], xs);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float es = exp2_fast(__builtin_fmaf(xs[j], c, -acc[0].r));
        acc[0].z += es;
        if constexpr (L1 == kL1Square) acc[2].z = __builtin_fmaf(es, es, acc[2].z);
        if constexpr (L1 == kL1Own) acc[2].z += exp2_fast(__builtin_fmaf(xs[j], kLog2e, -acc[2].r));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  {
    constexpr float kBig = 1.2676506e30f;  // 2^100
    bool odd = !(acc[0].z < kBig);
    if constexpr (LSE1) odd = odd || !(acc[2].z < kBig);
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {  // wave-uniform
      acc[0].init();
      acc[2].init();
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (mine(k)) {
          float xs[8];
          unpack8(sreg[k], xs);
          acc[0].add8(xs, c);
          if constexpr (LSE1) acc[2].add8(xs, kLog2e);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // the conversions stay here: behind the sums, and in front of this workgroup's post (rows in place)
  asm volatile("" : "+v"(s_y_bits), "+v"(sup_first), "+v"(s_e_bits));
  const float s_y = bf16_lo(s_y_bits);
  if (last && tid < n_edge) {
    const float xs = bf16_lo(s_e_bits);
    acc[0].add1(xs, c);
    if constexpr (LSE1) acc[2].add1(xs, kLog2e);
  }

  // ---- the teacher's normaliser over the k values, the range check of the ids, the gathered support logits
  Lse tt;
  tt.init();
  int bad_index = 0;
  auto each_entry = [&](auto&& f) {
    if (has_entry) f(tid, id_first, v_first);
    for (int j = tid + TH; j < k_top; j += TH) f(j, irow[j], vrow[j]);
  };
  each_entry([&](int j, int id, float v) {
    tt.add1(v, c);
    if ((unsigned)id >= (unsigned)V) bad_index = 1;
    if (needs(id)) sup_s[j] = j == tid ? (uint16_t)sup_first : srow[id];
  });

  // ---- wave totals, workgroup totals, post, wait, row totals (student); workgroup totals of the teacher's k values
  const int lane = tid & (kWave - 1), wid = tid / kWave;
  Lse st[2] = {acc[0], acc[2]};
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    normalise(st[i]);
    wave_merge_rescaled<false>(st[i]);
  }
  normalise(tt);
  wave_merge_rescaled<false>(tt);
  bad_index = __builtin_amdgcn_ballot_w64(bad_index != 0) != 0;
  if constexpr (NWV == 1) row_sync<TH>();  // the gathered support logits before their readers
  if constexpr (NWV > 1) {
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        red[(i * 2 + 0) * NWV + wid] = st[i].r;
        red[(i * 2 + 1) * NWV + wid] = st[i].z;
      }
      red[4 * NWV + wid] = tt.r;
      red[5 * NWV + wid] = tt.z;
      red[6 * NWV + wid] = bad_index ? 1.0f : 0.0f;
    }
    __syncthreads();  // also orders the gathered support logits in sup_s before their readers
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      st[i].init();
      if (lane < NWV) {
        st[i].r = red[(i * 2 + 0) * NWV + lane];
        st[i].z = red[(i * 2 + 1) * NWV + lane];
      }
      wave_merge_rescaled<false, merge_lanes(NWV)>(st[i]);
    }
    tt.init();
    if (lane < NWV) {
      tt.r = red[4 * NWV + lane];
      tt.z = red[5 * NWV + lane];
    }
    wave_merge_rescaled<false, merge_lanes(NWV)>(tt);
    bad_index = __builtin_amdgcn_ballot_w64(lane < NWV && red[6 * NWV + (lane & (NWV - 1))] != 0.0f) != 0;  // uniform
  }

  bool timeout = false;
  if constexpr (!SOLO) {
    const size_t abandon = (size_t)gridDim.x * W;  // behind the record
    if (tid < NW3) {
      float v = st[0].r;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        if (tid == i * 3 + 0) v = st[i].r;
        if (tid == i * 3 + 1) v = st[i].z;
        if (tid == i * 3 + 2) v = 0.0f;
      }
      gang_post(a.ws, (size_t)blockIdx.x * W + tid, v, a.tag);
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
    for (int i = 0; i < NS; ++i) {
      st[i].init();
      if (lane < G) {
        st[i].r = __builtin_bit_cast(float, xch[lane * W + i * 3 + 0]);
        st[i].z = __builtin_bit_cast(float, xch[lane * W + i * 3 + 1]);
      }
      if (G <= 16)  // uniform
        wave_merge_rescaled<false, 16>(st[i]);
      else
        wave_merge_rescaled<false>(st[i]);
    }
  }

  const float Ls = st[0].log2_sum();
  const float Lt = tt.log2_sum();
  const float lse1_s = __fmul_rn(LSE1 ? st[1].log2_sum() : Ls, kLn2);
  const bool ce = a.cscale != 0.0f;  // uniform
  Sweep2Coef kf = sweep2_coef(st[0], tt, st[NS - 1], c, a.gscale, a.cscale, true, false, LSE1);
  kf.folded = kf.folded && !a.ragged && !(SOLO && V < kCachedMinVocab);

  // ---- kd_tok (slice 0) and the final values of the support positions of this slice
  float part_kd = 0.0f;
  int y_hit = 0;
  if (!bad_index) {
    each_entry([&](int j, int id, float v) {
      const int at = place(id);
      if (slice == 0 || at >= 0) {
        const float b = v * c;
        const float sj = bf16_one(sup_s[j]);
        if (slice == 0) {
          const float lpt = b - Lt;
          const float lps = __builtin_fmaf(sj, c, -Ls);
          part_kd = __builtin_fmaf(exp2_fast(lpt), __builtin_fmaxf(lpt - lps, -3.4028234663852886e38f) * kLn2, part_kd);
        }
        if (GRAD && at >= 0) {
          float gj = grad_pair_elem(sj, b, kf.p);
          if (ce && id == y) {
            gj -= a.cscale;
            y_hit = 1;
          }
          sup_s[j] = one_bf16(gj);  // this thread read sup_s[j] above: no other thread touches entry j before the barrier
          link[j] = atomicExch(&first[at], (uint32_t)(j + 1)) | ((uint32_t)((id - head) & 7) << 16);
        }
      }
    });
  }
  if constexpr (GRAD && NWV == 1) row_sync<TH>();  // the lists before their readers (else: the barrier below)
  float kd = wave_sum_dpp(part_kd);
  bool y_in_support = __builtin_amdgcn_ballot_w64(y_hit != 0) != 0;  // the label is one of the support positions
  if constexpr (NWV > 1) {
    if constexpr (SOLO) __syncthreads();  // the first merge's readers of `red` are done
    if (lane == 0) {
      red[wid] = kd;
      if (y_in_support) y_hit_row = 1;
    }
    __syncthreads();
    y_in_support = y_hit_row != 0;
    if constexpr (NWV == 4)
      kd = (red[0] + red[1]) + (red[2] + red[3]);
    else
      kd = wave_sum_dpp(lane < NWV ? red[lane] : 0.0f);
  }
  kd = kd < 0.0f ? 0.0f : kd;
  if (bad_index) kd = __builtin_nanf("");

  if (tid == 0) {
    const float nanv = __builtin_nanf("");
    int flags = 0;
    if (slice == 0) {
      if (timeout) flags |= 8;
      if (bad_index) flags |= 2;
      if (bad_label && (a.nll || ce)) flags |= 1;
      if (a.kd) a.kd[row] = timeout ? nanv : kd;
      if (a.lse) a.lse[row] = timeout ? nanv : lse1_s;
      if (bad_label && a.nll) a.nll[row] = nanv;
    } else if (timeout) {
      flags |= 8;
    }
    if (own_y && a.nll) a.nll[row] = timeout ? nanv : __fsub_rn(lse1_s, s_y);
    if (flags && a.status) atomicOr(a.status, flags);
  }

  if constexpr (!GRAD) return;
  // ---- sweep 2: dense part p_S * weights from the registers, the label's and the support positions' values put in, one store
  uint8_t* gslice = reinterpret_cast<uint8_t*>(grow + head) + (int64_t)first_group * 16;
  auto store = [&](int k, const uint4& o) {
    const u32x4 w = {o.x, o.y, o.z, o.w};
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(gslice + (size_t)k * (step * 16)) + tid);
  };
  if (timeout || bad_index || (ce && bad_label)) {  // uniform: the row cannot be differentiated
    const uint4 qnan = make_uint4(0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (mine(k)) store(k, qnan);
    if (last && tid < n_edge) grow[sp.edge_elem(tid)] = 0x7fc0;
    return;
  }
  // the label position of the composite loss, unless it is one of the support positions (put in with them)
  int k_y = -1;
  uint4 y_keep = make_uint4(~0u, ~0u, ~0u, ~0u), y_bits = make_uint4(0, 0, 0, 0);
  uint16_t y_tail = 0;
  const bool patch_y = ce && own_y && !y_in_support;  // uniform
  if (patch_y) {
    const uint32_t b16 = one_bf16(grad_student_elem(s_y, kf.p) - a.cscale);
    y_tail = (uint16_t)b16;
    if (place_y < K * TH) {
      k_y = place_y / TH;
      if (place_y % TH == tid) {
        const int j = (y - head) & 7;
        const uint32_t keep = (j & 1) ? 0x0000ffffu : 0xffff0000u, bits = (j & 1) ? b16 << 16 : b16;
        if ((j >> 1) == 0) { y_keep.x = keep; y_bits.x = bits; }
        if ((j >> 1) == 1) { y_keep.y = keep; y_bits.y = bits; }
        if ((j >> 1) == 2) { y_keep.z = keep; y_bits.z = bits; }
        if ((j >> 1) == 3) { y_keep.w = keep; y_bits.w = bits; }
      }
    }
  }
  auto patch_label = [&](uint4& o) {
    o.x = (o.x & y_keep.x) | y_bits.x;
    o.y = (o.y & y_keep.y) | y_bits.y;
    o.z = (o.z & y_keep.z) | y_bits.z;
    o.w = (o.w & y_keep.w) | y_bits.w;
  };
  // the final values of the support positions on the list that begins with entry j1 - 1
  auto patch_support = [&](uint4& o, uint32_t j1) {
    while (j1 != 0) {
      const uint32_t l = link[j1 - 1], b16 = sup_s[j1 - 1], e = l >> 16;
      j1 = l & 0xffffu;
      const uint32_t keep = (e & 1) ? 0x0000ffffu : 0xffff0000u, bits = (e & 1) ? b16 << 16 : b16;
      o.x = (e >> 1) == 0 ? (o.x & keep) | bits : o.x;
      o.y = (e >> 1) == 1 ? (o.y & keep) | bits : o.y;
      o.z = (e >> 1) == 2 ? (o.z & keep) | bits : o.z;
      o.w = (e >> 1) == 3 ? (o.w & keep) | bits : o.w;
    }
  };
  auto walk = [&](auto form) {
    constexpr int FORM = decltype(form)::value;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
      if (mine(k)) {
        opaque(sreg[k]);
        uint4 o = grad8<kTopk, FORM>(sreg[k], sreg[k], kf);
        if (k == k_y) patch_label(o);  // uniform
        patch_support(o, first[k * TH + tid]);
        store(k, o);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (LSE1 && ce)  // uniform
    walk(std::integral_constant<int, L1 == kL1Square ? kPreciseCeSquare : kPreciseCeOwn>{});
  else if (kf.folded)
    walk(std::integral_constant<int, kFolded>{});
  else if (ce)
    walk(std::integral_constant<int, kPreciseCe>{});
  else
    walk(std::integral_constant<int, kPrecise>{});
  if (last && tid < n_edge) {
    const int e = sp.edge_elem(tid);
    uint16_t o = one_bf16(grad_student_elem(bf16_lo(s_e_bits), kf.p));
    if (patch_y && e == y) o = y_tail;
    const uint32_t j1 = first[K * TH + tid];
    if (j1 != 0) o = sup_s[j1 - 1];
    grow[e] = o;
  }
}

}  // namespace npd
