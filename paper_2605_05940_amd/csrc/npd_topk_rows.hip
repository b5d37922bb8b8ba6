// Teacher-side top-k record of rows that fit one workgroup's registers (up to 16,384 logits, k <= 256), at any offset
// from a 16-byte boundary.  Same exact selection and the same record as npd_topk_kernels.hip.
//
// Such rows were bound by the serial phases of a workgroup of 512 or 1024 threads per row (a sort of the thread maxima,
// block-wide counting, 20 barriers) with one read or two of the row in front: 65,536 rows of 1,024 .. 8,192 logits took
// 0.6 .. 1.6 ms for k = 64, 1 .. 23 % of the HBM peak.  Here a row belongs to TH threads that hold K groups of eight logits each (one
// wave for up to 4,096 logits, without a single barrier; four such rows share a workgroup), and the bound that picks the
// candidates is taken from the maxima of the groups, not of the threads: the k-th largest of them (each wave's
// ceil(k / waves)-th, the smallest report of all waves) lets barely more than k elements through, so the list that
// has to be ordered is short -- rank sort, all pairs, 32-bit words.  Where k is most of the groups or more, and
// where more elements pass than the list holds (massive ties), the k-th key itself is found by bisection over the
// registers and the ties are taken in id order.
#include "npd_kd_gang.hpp"
#include "npd_topk_order.hpp"

namespace npd {

namespace {

constexpr int kRowsTopkMax = 256;   // largest k
constexpr int kRowsCand = 512;      // candidates a row's list holds

// candidate word: larger = better (16-bit key, then the smaller id); ids are below 65,536 here
__device__ __forceinline__ uint32_t row_word(int o, int id) { return (key_of_ordered(o) << 16) | (0xffffu - (uint32_t)id); }

template <int TH>
struct RowTopkShared {
  __attribute__((aligned(16))) uint32_t cand[kRowsCand];
  uint32_t sorted[kRowsTopkMax];
  int ncand;
  int red[TH / kWave];
  float fred[TH / kWave];
};

template <int TH>
__device__ __forceinline__ void rows_sync() {
  if constexpr (TH == kWave)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  else
    __syncthreads();
}

// sum over the TH threads of a row
template <int TH>
__device__ __forceinline__ int rows_sum(int v, int* red) {
  if constexpr (TH == kWave) return (int)wave_sum_dpp((float)v);  // (whole numbers below 2^24)
  return block_sum_int<TH>(v, red);
}

// exclusive prefix over the TH threads of a row, in thread order, and the total
template <int TH>
__device__ __forceinline__ int rows_scan(int v, int* red, int tid, int& total) {
  const int lane = tid & (kWave - 1), wid = tid / kWave;
  int incl = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int o = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += o;
  }
  int base = 0;
  total = __shfl(incl, kWave - 1, kWave);
  if constexpr (TH > kWave) {
    if (lane == kWave - 1) red[wid] = incl;
    __syncthreads();
    total = 0;
#pragma unroll
    for (int w = 0; w < TH / kWave; ++w) {
      if (w < wid) base += red[w];
      total += red[w];
    }
    __syncthreads();
  }
  return base + incl - v;
}

}  // namespace

template <int TH, int K>
__global__ __launch_bounds__(TH == kWave ? 4 * TH : TH, K <= 4 ? 8 : 5) void teacher_topk_row_kernel(const TopkArgs a) {
  constexpr int ROWS = TH == kWave ? 4 : 1;
  constexpr int NW = TH / kWave;
  __shared__ RowTopkShared<TH> shs[ROWS];
  const int tid = threadIdx.x % (unsigned)TH, lane = tid & (kWave - 1), wid = tid / kWave;
  const int sub = ROWS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / TH);
  RowTopkShared<TH>& sh = shs[sub];
  const int64_t row = (int64_t)blockIdx.x * ROWS + sub;
  if (ROWS > 1 && row >= a.T) return;
  const int V = a.V, k = a.k;
  int32_t* irow = a.idx + row * (int64_t)k;
  float* vrow = a.val + row * (int64_t)k;
  if (a.mask && !a.mask[row]) {  // not scored: a harmless record (valid ids, zero values)
    for (int j = tid; j < k; j += TH) {
      irow[j] = j;
      vrow[j] = 0.0f;
    }
    return;
  }
  const uint16_t* trow = a.t + row * a.stride;
  const RowSplit sp = row_split(trow, V, true);
  const int head = sp.head, nvec = sp.nvec, n_edge = V - nvec * 8;
  if (tid == 0) sh.ncand = 0;

  // ---- the row, as ordered 16-bit integers (value order, -0 directly below +0)
  const __amdgpu_buffer_rsrc_t rt = row_rsrc(trow + head, nvec);
  const int n_mine = (nvec - tid + TH - 1) / TH;  // groups of this thread
  uint4 g[K];
#pragma unroll
  for (int i = 0; i < K; ++i) g[i] = ld_group<TH * 16>(rt, tid * 16, i, true, true);
  int edge = -32768;  // this thread's edge element
  if (tid < n_edge) edge = ordered_of(trow[sp.edge_elem(tid)]);
  int gmax[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    g[i] = make_uint4(pk_ordered(g[i].x), pk_ordered(g[i].y), pk_ordered(g[i].z), pk_ordered(g[i].w));
    const short2v m = pk_max(pk_max(as_s2(g[i].x), as_s2(g[i].y)), pk_max(as_s2(g[i].z), as_s2(g[i].w)));
    gmax[i] = i < n_mine ? max((int)m.x, (int)m.y) : -32768;  // below every element
  }
  auto element = [&](int i, int j) -> int {  // i, j compile-time after unrolling
    const uint32_t d = (j >> 1) == 0 ? g[i].x : (j >> 1) == 1 ? g[i].y : (j >> 1) == 2 ? g[i].z : g[i].w;
    return (j & 1) ? (int)d >> 16 : (int)(short)(uint16_t)d;
  };
  auto id_of = [&](int i, int j) { return head + (i * TH + tid) * 8 + j; };
  auto append = [&](int o, int id) {
    const int pos = atomicAdd(&sh.ncand, 1);
    if (pos < kRowsCand) sh.cand[pos] = row_word(o, id);
  };

  // ---- the bound: each wave's m-th largest group maximum; NW m >= k elements of the row are >= the smallest report.
  // Every wave owns at least (nvec / TH) * 64 whole groups.
  const int m = (k + NW - 1) / NW;
  // Beyond three quarters of a wave's maxima the bound lets more than 1.7 k elements through.
  bool exact = m > nvec / TH * kWave / 4 * 3;  // uniform
  if (!exact) {
    int lmax = gmax[0], lmin = gmax[0];
#pragma unroll
    for (int i = 1; i < K; ++i) {
      lmax = max(lmax, gmax[i]);
      lmin = min(lmin, gmax[i]);
    }
    int bhi = lmax, blo = m <= kWave ? lmax : lmin;  // count(maxima >= blo) >= m: a maximum per lane, or all of them
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      bhi = max(bhi, __shfl_xor(bhi, off, kWave));
      blo = min(blo, __shfl_xor(blo, off, kWave));
    }
    bhi = __builtin_amdgcn_readfirstlane(bhi) + 1;  // count(maxima >= bhi) = 0
    blo = __builtin_amdgcn_readfirstlane(blo);
    while (bhi - blo > 1) {
      const int mid = (blo + bhi) >> 1;
      int n = 0;
#pragma unroll
      for (int i = 0; i < K; ++i) n += __popcll(__ballot(gmax[i] >= mid));
      if (n >= m)
        blo = mid;
      else
        bhi = mid;
    }
    int L = blo;
    if constexpr (NW > 1) {
      if (lane == 0) sh.red[wid] = blo;
      __syncthreads();  // also orders ncand = 0 before the first append
#pragma unroll
      for (int w = 0; w < NW; ++w) L = min(L, sh.red[w]);
    } else {
      rows_sync<TH>();
    }
    const int Lp = L == 0 ? -1 : L;  // +0 and -0 are one value
#pragma unroll
    for (int i = 0; i < K; ++i) {
      if (gmax[i] >= Lp && i < n_mine) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int o = element(i, j);
          if (o >= Lp) append(o, id_of(i, j));
        }
      }
    }
    if (tid < n_edge && edge >= Lp) append(edge, sp.edge_elem(tid));
    rows_sync<TH>();
    exact = sh.ncand > kRowsCand;
  } else {
    rows_sync<TH>();
  }
  int n = sh.ncand;
  if (exact) {
    // ---- the k-th key by bisection over the registers, then the ties at it in id order
    rows_sync<TH>();
    if (tid == 0) sh.ncand = 0;
    auto canonical = [](int o) { return o == -1 ? 0 : o; };  // -0 is +0
    int lo = -32768, hi = 32768;  // count(>= lo) >= k, count(>= hi) < k
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      int c = tid < n_edge && canonical(edge) >= mid;
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (i < n_mine) {
#pragma unroll
          for (int j = 0; j < 8; ++j) c += canonical(element(i, j)) >= mid;
        }
      c = rows_sum<TH>(c, sh.red);
      if (c >= k)
        lo = mid;
      else
        hi = mid;
    }
    const int Tk = lo;
    rows_sync<TH>();
    int above = 0;  // fewer than k <= kRowsCand of them
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (i < n_mine) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int o = canonical(element(i, j));
          if (o > Tk) {
            ++above;
            append(o, id_of(i, j));
          }
        }
      }
    if (tid < n_edge && canonical(edge) > Tk) {
      ++above;
      append(edge, sp.edge_elem(tid));
    }
    above = rows_sum<TH>(above, sh.red);
    rows_sync<TH>();
    const int need = k - above;  // ties to take, lowest ids first (>= 1)
    int taken = 0;               // uniform
    auto take = [&](int mine, auto&& put) {  // `mine` ties of this thread, in thread order behind the ones taken so far
      int total;
      const int rank = taken + rows_scan<TH>(mine, sh.red, tid, total);
      if (mine && rank < need) put(rank);
      taken += total;
    };
    const bool edge_tie = tid < n_edge && canonical(edge) == Tk;
    auto put_edge = [&](int rank) { sh.cand[above + rank] = row_word(edge, sp.edge_elem(tid)); };
    take(edge_tie && tid < head, put_edge);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      int mine = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) mine += i < n_mine && canonical(element(i, j)) == Tk;
      take(mine, [&](int rank) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (canonical(element(i, j)) == Tk) {
            if (rank < need) sh.cand[above + rank] = row_word(Tk, id_of(i, j));
            ++rank;
          }
      });
    }
    take(edge_tie && tid >= head, put_edge);
    rows_sync<TH>();
    n = k;
  }

  // ---- rank sort: the rank of a word is the number of larger words (all distinct)
  const int n4 = (n + 3) / 4;
  if (tid < n4 * 4 - n) sh.cand[n + tid] = 0;  // below every candidate (n <= kRowsCand, a multiple of 4)
  rows_sync<TH>();
  for (int i = tid; i < n; i += TH) {
    const uint32_t w = sh.cand[i];
    int r = 0;
    for (int j = 0; j < n4; ++j) {
      const uint4 x = reinterpret_cast<const uint4*>(sh.cand)[j];
      r += (x.x > w) + (x.y > w) + (x.z > w) + (x.w > w);
    }
    if (r < k) sh.sorted[r] = w;
  }
  rows_sync<TH>();
  float lse = 0.0f;
  if (a.log_probs) {  // log-softmax over the k selected logits; the first one is the largest
    const float v0 = value_of_key(sh.sorted[0] >> 16);
    float part = 0.0f;
    for (int j = tid; j < k; j += TH) part += __expf(value_of_key(sh.sorted[j] >> 16) - v0);
    part = TH == kWave ? wave_sum(part) : block_sum<TH>(part, sh.fred);
    lse = v0 + __logf(part);
  }
  for (int j = tid; j < k; j += TH) {
    const uint32_t w = sh.sorted[j];
    irow[j] = (int32_t)(0xffffu - (w & 0xffffu));
    vrow[j] = value_of_key(w >> 16) - lse;
  }
}

template <int TH, int K>
static hipError_t launch_rows(const TopkArgs& a, hipStream_t stream) {
  constexpr int ROWS = TH == kWave ? 4 : 1;
  return launch_kernel(teacher_topk_row_kernel<TH, K>, dim3((unsigned)((a.T + ROWS - 1) / ROWS)), dim3(TH * ROWS), 0,
                       stream, a);
}

// Measured (MI355X, 65,536 rows -- 61,035 of 16,384 logits, 40,690 of 24,576 --, all scored, us; the kernels of
// npd_topk_kernels.hip / this one): k = 64 V = 1,024 1,594 / 91, 4,096 1,579 / 179, 8,192 586 / 274, 16,384 616 / 449,
// 24,576 463 / 683; k = 10 1,486 / 48, 1,480 / 99, 467 / 180, 490 / 329, 360 / 544.  Longer rows are better off with the kernel that streams them: eight waves that wait
// for one another at every step no longer hide behind other rows.
// Few rows do not hide a row's serial steps behind others: they stay with the kernels of 512 or 1024 threads per row
// where the list to order is long or most of the row (T = 64, V = 2,500: k = 20 11.0 / 6.4 us, 64 11.6 / 10.5, 128
// 12.9 / 16.2).
constexpr int kManyRows = 1024;
bool topk_rows_applies(const TopkArgs& a) {
  if (a.k > kRowsTopkMax || a.V / 8 > 256 * 8) return false;
  return a.T >= kManyRows || (a.k <= 64 && 16 * a.k <= a.V);
}

hipError_t launch_topk_rows(const TopkArgs& a, hipStream_t stream) {
  const int nvec = a.V / 8;
  if (nvec <= 64 * 2) return launch_rows<64, 2>(a, stream);
  if (a.T < kManyRows) {  // more threads per row
    if (nvec <= 128 * 2) return launch_rows<128, 2>(a, stream);
    if (nvec <= 256 * 2) return launch_rows<256, 2>(a, stream);
    if (nvec <= 256 * 4) return launch_rows<256, 4>(a, stream);
    return launch_rows<256, 8>(a, stream);
  }
  if (nvec <= 64 * 4) return launch_rows<64, 4>(a, stream);
  if (nvec <= 64 * 8) return launch_rows<64, 8>(a, stream);
  if (nvec <= 128 * 8) return launch_rows<128, 8>(a, stream);
  return launch_rows<256, 8>(a, stream);
}

}  // namespace npd
