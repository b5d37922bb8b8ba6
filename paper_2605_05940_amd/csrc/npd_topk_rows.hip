// Teacher-side top-k record of rows that fit one workgroup's registers (up to 65,536 logits, k <= 256), at any offset
// from a 16-byte boundary.  Same exact selection and the same record as npd_topk_kernels.hip.
//
// A row belongs to TH threads that hold K groups of eight logits each (one wave for up to 4,096 logits, without a single
// barrier; four such rows share a workgroup).  The bound that picks the candidates is taken from maxima of the row's
// parts, as fine as k asks for, so that barely more than k elements pass; the groups that hold one are staged and looked
// at 64 at a time, one to a lane; one wave then orders the list in its registers.  What bounds such rows is the vector
// instructions of these serial steps, not the bytes.  Measured (MI355X, all scored, us; candidates appended one by one through
// an atomic counter and ranked by comparing all pairs / this; k = 10, 64, 256):
//   32,768 rows of 1,024   25.3 / 22.9, 47.2 / 36.2, 177 / 85      8,192 rows of 8,192  27.4 / 22.9, 42.3 / 30.2, 106 / 52
//   32,768 rows of 16,384  175 / 163 (6.6 TB/s), 246 / 164, 524 / 283
// Where k is most of the row's pairs, and where more elements pass than the list holds (massive ties), the k-th key
// itself is found by bisection over the registers and the ties are taken in id order.
#include "npd_kd_gang.hpp"
#include "npd_topk_order.hpp"

namespace npd {

namespace {

constexpr int kRowsTopkMax = 256;   // largest k
// candidates a row's list holds: with more waves each wave's bound is a smaller sample's (300 rows of 50,304 normal
// logits, k = 256, 16 waves: 481 candidates on average, 717 at most; 4 waves, 16,384 logits: 328 and 433)
constexpr int rows_cand(int th) { return th >= 256 ? 2 * kWaveSortMax : kWaveSortMax; }

constexpr int kRowsStage = 2 * kWave;  // groups with a candidate that a wave stages before it looks at their elements
constexpr int kRowsMaxVocab = 1 << 16;
constexpr CandWord kRowsWord{0u, 16};  // ids below 65,536: a candidate is one 32-bit word whatever the keys
__device__ __forceinline__ uint32_t rows_word(int o, int id) { return kRowsWord.make(key_of_ordered(o), (uint32_t)id); }

template <int TH>
struct RowTopkShared {
  uint4 group[TH / kWave][kRowsStage];
  uint32_t cand[rows_cand(TH)];
  int group_id[TH / kWave][kRowsStage];
  int ncand;
  int red[TH / kWave];
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
__global__ __launch_bounds__(TH == kWave ? 4 * TH : TH, TH == 1024 ? 4 : K <= 4 && TH < 512 ? 8 : 5) void teacher_topk_row_kernel(const TopkArgs a) {
  constexpr int ROWS = TH == kWave ? 4 : 1;
  constexpr int NW = TH / kWave, kRowsCand = rows_cand(TH);
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
  auto group_max = [&](int i) -> int {
    const short2v m = pk_max(pk_max(as_s2(g[i].x), as_s2(g[i].y)), pk_max(as_s2(g[i].z), as_s2(g[i].w)));
    return i < n_mine ? max((int)m.x, (int)m.y) : -32768;  // below every element
  };
  int lmax = -32768, lmin = 32767;  // largest and smallest maximum of this thread's groups
#pragma unroll
  for (int i = 0; i < K; ++i) {
    g[i] = make_uint4(pk_ordered(g[i].x), pk_ordered(g[i].y), pk_ordered(g[i].z), pk_ordered(g[i].w));
    const int x = group_max(i);
    lmax = max(lmax, x);
    if (i < n_mine) lmin = min(lmin, x);
  }
  auto element = [&](int i, int j) -> int {  // i, j compile-time after unrolling
    const uint32_t d = (j >> 1) == 0 ? g[i].x : (j >> 1) == 1 ? g[i].y : (j >> 1) == 2 ? g[i].z : g[i].w;
    return (j & 1) ? (int)d >> 16 : (int)(short)(uint16_t)d;
  };
  auto id_of = [&](int i, int j) { return head + (i * TH + tid) * 8 + j; };
  auto append = [&](int o, int id) {
    const int pos = atomicAdd(&sh.ncand, 1);
    if (pos < kRowsCand) sh.cand[pos] = rows_word(o, id);
  };

  // ---- the bound: each wave's m-th largest of some maxima of its elements; NW m >= k elements of the row are >= the
  // smallest report.  Maxima of finer parts give a bound that fewer elements pass and take longer to bisect: one per thread
  // where m is at most a quarter of them (1.15 k elements pass), one per group up to half (1.4 k), one per pair of elements
  // up to three quarters (1.2 .. 1.4 k); every wave owns at least `units` whole groups.
  const int m = (k + NW - 1) / NW;
  const int units = NW == 1 ? nvec : nvec / TH * kWave;
  const bool per_thread = 4 * m <= kWave && units >= kWave, per_group = 2 * m <= units;  // uniform
  constexpr bool kFine = K <= 8;  // (registers)
  bool exact = kFine ? m > 3 * units : !per_thread;  // uniform
  if (!exact) {
    int bhi = lmax, blo = per_thread ? lmax : lmin;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      bhi = max(bhi, __shfl_xor(bhi, off, kWave));
      blo = min(blo, __shfl_xor(blo, off, kWave));
    }
    bhi = __builtin_amdgcn_readfirstlane(bhi) + 1;  // count(maxima >= bhi) = 0
    blo = __builtin_amdgcn_readfirstlane(blo);
    int bound;
    if (per_thread || !kFine) {
      const int x[1] = {lmax};
      bound = wave_bound(x, m, m / 8, blo, bhi);
    } else if (per_group) {
      int gmax[K];
#pragma unroll
      for (int i = 0; i < K; ++i) gmax[i] = group_max(i);
      bound = wave_bound(gmax, m, m / 8, blo, bhi);
    } else {
      int pmax[4 * K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) pmax[4 * i + j] = i < n_mine ? max(element(i, 2 * j), element(i, 2 * j + 1)) : -32768;
      }
      bound = wave_bound(pmax, m, m / 8, -32768, bhi);
    }
    int L = bound;
    if constexpr (NW > 1) {
      if (lane == 0) sh.red[wid] = bound;
      __syncthreads();  // also orders ncand = 0 before the first append
#pragma unroll
      for (int w = 0; w < NW; ++w) L = min(L, sh.red[w]);
    } else {
      rows_sync<TH>();
    }
    const int Lp = L == 0 ? -1 : L;  // +0 and -0 are one value
    // ---- the groups with an element >= Lp are staged whole, up to 64 of them are then looked at together, one to a lane
    uint4* sgroup = sh.group[wid];
    int* sid = sh.group_id[wid];
    int staged = 0, listed = 0;  // uniform; `listed`: candidates of this wave (one wave per row: of the row)
    auto look = [&](int count) {  // at the last `count` <= 64 staged groups
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
      const int at = staged - count + lane;
      uint4 v = make_uint4(0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u);
      int id0 = 0;
      if (lane < count) {
        v = sgroup[at];
        id0 = head + sid[at] * 8;
      }
      auto elem = [&](int j) -> int {
        const uint32_t d = (j >> 1) == 0 ? v.x : (j >> 1) == 1 ? v.y : (j >> 1) == 2 ? v.z : v.w;
        return (j & 1) ? (int)d >> 16 : (int)(short)(uint16_t)d;
      };
      int mine = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) mine += lane < count && elem(j) >= Lp;
      const int incl = wave_scan(mine);
      const int total = __builtin_amdgcn_readlane(incl, 63);
      int base = listed;
      if constexpr (NW > 1) {
        if (lane == 0) base = atomicAdd(&sh.ncand, total);
        base = __builtin_amdgcn_readfirstlane(base);
      }
      listed += total;
      int pos = base + incl - mine;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (lane < count && elem(j) >= Lp) {
          if (pos < kRowsCand) sh.cand[pos] = rows_word(elem(j), id0 + j);
          ++pos;
        }
      }
      staged -= count;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    };
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const bool pass = group_max(i) >= Lp && i < n_mine;
      const unsigned long long who = __ballot(pass);
      if (pass) {
        const int at = staged + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
        sgroup[at] = g[i];
        sid[at] = i * TH + tid;
      }
      staged += __popcll(who);  // (fewer than 64 before)
      if (staged >= kWave) look(kWave);
    }
    if (staged > 0) look(staged);
    if constexpr (NW == 1) {
      if (lane == 0) sh.ncand = listed;
      rows_sync<TH>();
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
    auto put_edge = [&](int rank) { sh.cand[above + rank] = rows_word(edge, sp.edge_elem(tid)); };
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
            if (rank < need) sh.cand[above + rank] = rows_word(Tk, id_of(i, j));
            ++rank;
          }
      });
    }
    take(edge_tie && tid >= head, put_edge);
    rows_sync<TH>();
    n = k;
  }

  // ---- one wave orders the list in its registers
  if (wid == 0) {
    uint32_t* cand = sh.cand;
    wave_order_and_emit_any([&](int i) { return cand[i]; }, n, k, kRowsWord, cand, a.log_probs, irow, vrow, lane);
  }
}

template <int TH, int K>
static hipError_t launch_rows(const TopkArgs& a, hipStream_t stream) {
  constexpr int ROWS = TH == kWave ? 4 : 1;
  return launch_kernel(teacher_topk_row_kernel<TH, K>, dim3((unsigned)((a.T + ROWS - 1) / ROWS)), dim3(TH * ROWS), 0,
                       stream, a);
}

// Which rows.  Longer rows are better off with the kernels that stream them unless there are so few that each has a compute
// unit (1,024 threads) or half of one (512 threads) to itself and waits for its own latency.  Measured (MI355X, all
// scored, us, streamed / this): 256 rows of 50,304 k = 10 10.0 / 9.7, 64 11.1 / 10.4, 256 17.4 / 14.1; 400 rows of 32,000
// k = 10 10.2 / 9.5, 256 15.6 / 13.9; 600 of 32,000 11.7 / 12.9, 19.3 / 22.8; 600 of 18,000 9.7 / 12.0, 15.7 / 21.5; 400 of
// 18,000 8.7 / 8.6, 13.8 / 14.0.
constexpr int kManyRows = 1024;
bool topk_rows_applies(const TopkArgs& a) {
  const int nvec = a.V / 8;
  if (a.k > kRowsTopkMax || a.V > kRowsMaxVocab) return false;
  if (nvec <= 256 * 8) return true;
  if (nvec <= 512 * 8) return a.T <= 2 * kTopkFewRows;
  return a.T <= kTopkFewRows;
}

hipError_t launch_topk_rows(const TopkArgs& a, hipStream_t stream) {
  const int nvec = a.V / 8;
  if (nvec <= 64 * 2) return launch_rows<64, 2>(a, stream);
  if (nvec > 512 * 8) return launch_rows<1024, 8>(a, stream);
  if (nvec > 256 * 8 || (nvec > 256 * 4 && a.k > 64 && a.T <= kManyRows / 2)) return launch_rows<512, 8>(a, stream);
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
