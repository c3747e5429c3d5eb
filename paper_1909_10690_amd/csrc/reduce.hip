// Reduction of one joint table per transform to Shannon MI (Eq. (1),
// Eq. (2)) and Tsallis MI for every requested q -- the same table serves
// every entropy (Discussion).  fp64 with compensated (Neumaier) partial
// sums per thread, wave64 shuffles and an ordered cross-wave combine, so
// the result does not depend on scheduling.
//
// One launch: a workgroup per (transform, row slice) forms the partial sums of
// its joint cells and of the marginals of its rows and of the same-numbered
// columns; the last workgroup of a transform to finish merges the slices in
// order.  Slicing spreads a single transform over up to B/8 CUs.  N comes with
// the table: the sweeps add it up as they flush.
//
// With p = h / N over the cells of X (N = total count or, for Parzen
// tables, the number of voxels that took part):
//   Shannon  H(X) = -sum p ln p,                MI = H(F) + H(M) - H(F,M)
//   Tsallis  S_q(X) = -sum p expm1((q-1) ln p) / (q-1)
//            I_q = S_q(F) + S_q(M) - S_q(F,M)  [+ (1-q) S_q(F) S_q(M), pseudo-additive]
// The expm1 form of (1 - sum p^q)/(q-1) keeps q near 1 free of cancellation.
#include "common.h"

#include <type_traits>

namespace gemi {

struct Comp {
  double s, c;
};

__device__ __forceinline__ void comp_add(Comp& a, double x) {
  const double t = a.s + x;
  if (fabs(a.s) >= fabs(x))
    a.c += (a.s - t) + x;
  else
    a.c += (x - t) + a.s;
  a.s = t;
}

// (s1, c1) + (s2, c2) with the rounding error of s1 + s2 kept (TwoSum).
__device__ __forceinline__ Comp comp_merge(Comp a, Comp b) {
  const double s = a.s + b.s;
  const double bb = s - a.s;
  const double err = (a.s - (s - bb)) + (b.s - bb);
  Comp r;
  r.s = s;
  r.c = a.c + b.c + err;
  return r;
}

// A line's sum: counts are summed in integers (N < 2^28), masses compensated.
template <bool TABLE>
struct LineSum;
template <>
struct LineSum<false> {
  uint32_t s;
  __device__ __forceinline__ void add(uint32_t x) { s += x; }
  __device__ __forceinline__ void merge_xor(int off) { s += __shfl_xor(s, off, 64); }
  __device__ __forceinline__ void merge(const LineSum& o) { s += o.s; }
  __device__ __forceinline__ double value() const { return (double)s; }
};
template <>
struct LineSum<true> {
  Comp a;
  __device__ __forceinline__ void add(double x) { comp_add(a, x); }
  __device__ __forceinline__ void merge_xor(int off) {
    Comp o;
    o.s = __shfl_xor(a.s, off, 64);
    o.c = __shfl_xor(a.c, off, 64);
    a = comp_merge(a, o);
  }
  __device__ __forceinline__ void merge(const LineSum& o) { a = comp_merge(a, o.a); }
  __device__ __forceinline__ double value() const { return a.s + a.c; }
};

// The wave's sums merged, in every lane: within rows of 16 lanes by DPP, then
// by the row and half swaps -- register moves, where a shuffle goes through
// LDS (24 round trips of which cost more than the sums themselves).  Merging
// is symmetric, so mirrored lanes serve as well as lanes an offset apart.
template <int DPP>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, DPP, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), DPP, 0xF, 0xF, true);
  return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}
template <int DPP>
__device__ __forceinline__ Comp dpp_merge(Comp a) {
  return comp_merge(a, Comp{dpp_f64<DPP>(a.s), dpp_f64<DPP>(a.c)});
}
// x: the lower (even row's, lower half's) value in both partners; y: the other
template <bool HALF>
__device__ __forceinline__ void swap_f64(double v, double& x, double& y) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t l = (uint32_t)u, h = (uint32_t)(u >> 32);
  const auto lo = HALF ? __builtin_amdgcn_permlane32_swap(l, l, false, false) : __builtin_amdgcn_permlane16_swap(l, l, false, false);
  const auto hi = HALF ? __builtin_amdgcn_permlane32_swap(h, h, false, false) : __builtin_amdgcn_permlane16_swap(h, h, false, false);
  x = __longlong_as_double((int64_t)(((uint64_t)hi[0] << 32) | lo[0]));
  y = __longlong_as_double((int64_t)(((uint64_t)hi[1] << 32) | lo[1]));
}
template <bool HALF>
__device__ __forceinline__ Comp swap_merge(Comp a) {
  Comp x, y;
  swap_f64<HALF>(a.s, x.s, y.s);
  swap_f64<HALF>(a.c, x.c, y.c);
  return comp_merge(x, y);
}
__device__ __forceinline__ Comp wave_merge(Comp a) {
  a = dpp_merge<0xB1>(a);   // quad_perm 1,0,3,2
  a = dpp_merge<0x4E>(a);   // quad_perm 2,3,0,1
  a = dpp_merge<0x141>(a);  // row_half_mirror
  a = dpp_merge<0x140>(a);  // row_mirror
  a = swap_merge<false>(a);
  return swap_merge<true>(a);
}

// Loads issued together per lane: a line's sum waits once for kLineLoads of
// them, not for each.
constexpr int kLineLoads = 8;
// Cells a thread takes at a time: more of them share a wave-wide merge where a
// slice has them.
constexpr int kCellsFew = 4, kCellsMany = 8;

// One workgroup per (transform, slice): per q, the compensated sums
//   joint  sum over the slice's cells of  f(p)
//   fixed  sum over the slice's rows of   f(row marginal)
//   moving sum over the slice's columns of f(column marginal)
// with f(p) = p ln p (Shannon) or p expm1((q-1) ln p) (Tsallis), p = h / N.
// What bounds it: for one transform, load latency and the fp64 chains of few
// waves (hence the batched loads, and one wave-wide merge per entropy for the
// cells and one for the marginals); for a thousand, the logarithms and
// exponentials of the occupied cells (ln p is taken once for all entropies).
// With the counts summed, the slices' sums formed and the slices merged by a
// kernel each: 44 us for one 128-bin table and six entropies, now 16; 168 us
// for 150 of 256 bins and two entropies, now 90.
template <bool TABLE, int CELLS>
__global__ __launch_bounds__(kBlock) void mi_reduce_kernel(ReduceLaunch L) {
  typedef typename std::conditional<TABLE, double, uint32_t>::type Cell;
  const int B = L.bins, S = L.splits, n_q = L.q.n;
  const int t = blockIdx.x / S, s = blockIdx.x - t * S;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* __restrict__ mi = L.mi_out + (size_t)t * n_q;
  int64_t Mq[12];
  const bool ok = quantize_transform(L.transforms + 12 * (size_t)t, Mq);
  // the upper half of the count is the slices' ticket; N < 2^28
  const uint32_t n_int = (uint32_t)__hip_atomic_load(&L.count[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!ok || n_int == 0) {  // a rejected matrix; no voxel took part
    if (s == 0) {
      if ((int)threadIdx.x < n_q) mi[threadIdx.x] = ok ? 0.0 : __longlong_as_double(0x7FF8000000000000ll);
      if (threadIdx.x == 0 && L.overlap_out) L.overlap_out[t] = 0;
    }
    return;
  }
  const double invN = 1.0 / (double)n_int;
  int r0, r1;
  slice_rows(B, S, s, r0, r1);
  const int R = r1 - r0;
  const size_t BB = (size_t)B * B;
  const Cell* __restrict__ h = (TABLE ? (const Cell*)L.table : (const Cell*)L.hist) + t * BB;
  const Cell* __restrict__ hs = h + (size_t)r0 * B;  // the slice's cells
  double* marg_out = L.marg_out ? L.marg_out + (size_t)t * 2 * B + r0 : nullptr;

  __shared__ double marg[512];  // marginals of the slice's rows (0..R-1) and columns (R..2R-1)
  __shared__ LineSum<TABLE> col[kBlock];
  // rows: lr lanes each, neighbouring lanes on neighbouring cells
  int lr = 8;
  while (lr < 64 && lr * R < kBlock) lr <<= 1;
  for (int l0 = 0; l0 < R; l0 += kBlock / lr) {
    const int r = l0 + (int)threadIdx.x / lr, sub = threadIdx.x & (lr - 1);
    LineSum<TABLE> a{};
    for (int k = sub; k < B; k += lr * kLineLoads) {
      Cell v[kLineLoads];
#pragma unroll
      for (int j = 0; j < kLineLoads; ++j) v[j] = r < R && k + j * lr < B ? hs[(size_t)r * B + k + j * lr] : (Cell)0;
#pragma unroll
      for (int j = 0; j < kLineLoads; ++j) a.add(v[j]);
    }
    for (int off = lr >> 1; off > 0; off >>= 1) a.merge_xor(off);
    if (sub == 0 && r < R) {
      marg[r] = a.value();
      if (marg_out) marg_out[r] = a.value();
    }
  }
  // columns: cw neighbouring ones at a time, kBlock / cw lanes each
  int cw = 8;
  while (cw < 64 && cw < R) cw <<= 1;
  const int groups = kBlock / cw, g = threadIdx.x / cw, cl = threadIdx.x & (cw - 1);
  for (int c0 = 0; c0 < R; c0 += cw) {
    const int c = c0 + cl;
    LineSum<TABLE> a{};
    for (int k = g; k < B; k += groups * kLineLoads) {
      Cell v[kLineLoads];
#pragma unroll
      for (int j = 0; j < kLineLoads; ++j)
        v[j] = c < R && k + j * groups < B ? h[(size_t)(k + j * groups) * B + r0 + c] : (Cell)0;
#pragma unroll
      for (int j = 0; j < kLineLoads; ++j) a.add(v[j]);
    }
    for (int off = cw; off < 64; off <<= 1) a.merge_xor(off);  // the wave's groups
    if (lane < cw) col[wave * cw + lane] = a;
    __syncthreads();
    if ((int)threadIdx.x < cw && c < R) {
      for (int w = 1; w < kBlock / 64; ++w) a.merge(col[w * cw + threadIdx.x]);
      marg[R + c] = a.value();
      if (marg_out) marg_out[B + c] = a.value();
    }
    __syncthreads();
  }

  // the cells, CELLS per thread at a time: p and ln p once, then per
  // entropy the thread's compensated sum, merged over the wave into its sum
  // per wave: cells; rows (even waves) or columns (odd)
  __shared__ Comp wpart[kMaxQ][kBlock / 64][2];
  for (int e = threadIdx.x; e < kMaxQ * (kBlock / 64) * 2; e += kBlock) (&wpart[0][0][0])[e] = Comp{0, 0};
  __syncthreads();
  // (an empty cell's sums are 0 without a branch, so that a thread's logarithms
  // and exponentials run side by side; with many cells, where a thousand
  // transforms keep the vector unit busy, the empty ones are skipped)
  auto entropies = [&]<int N>(const double (&x)[N], int slot) {
    double p[N], lp[N];
    bool any = false;
#pragma unroll
    for (int j = 0; j < N; ++j) any = any || x[j] > 0;
    if (__builtin_amdgcn_ballot_w64(any) == 0) return;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      p[j] = x[j] * invN;
      lp[j] = 0.0;
      if (N <= kCellsFew || x[j] > 0) lp[j] = log(x[j] > 0 ? p[j] : 1.0);
    }
    for (int iq = 0; iq < n_q; ++iq) {
      const double qm1 = L.q.q[iq] - 1.0;
      Comp a = {0, 0};
      if (qm1 == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) comp_add(a, p[j] * lp[j]);
      } else {
        double f[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
          f[j] = 0.0;
          if (N <= kCellsFew || x[j] > 0) f[j] = p[j] * expm1(qm1 * lp[j]);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) comp_add(a, f[j]);
      }
      a = wave_merge(a);
      if (lane == 0) wpart[iq][wave][slot] = comp_merge(wpart[iq][wave][slot], a);
    }
  };
  const int nc = R * B;
  for (int e0 = 0; e0 < nc; e0 += kBlock * CELLS) {
    double x[CELLS];
#pragma unroll
    for (int j = 0; j < CELLS; ++j) {
      const int e = e0 + j * kBlock + (int)threadIdx.x;
      x[j] = e < nc ? (double)hs[e] : 0.0;
    }
    entropies(x, 0);
  }
  // even waves the rows' marginals, odd ones the columns'
  for (int e0 = 64 * (wave >> 1); e0 < R; e0 += 64 * (kBlock / 128)) {
    const double x[1] = {e0 + lane < R ? marg[(wave & 1 ? R : 0) + e0 + lane] : 0.0};
    entropies(x, 1);
  }
  __syncthreads();
  if (wave != 0) return;

  // lane 3 iq + k: sum k (joint, fixed, moving) of entropy iq
  const int iq = lane / 3, k = lane - 3 * iq;
  Comp tot = {0, 0};
  if (iq < n_q) {
    const int w0 = k == 2 ? 1 : 0, step = k == 0 ? 1 : 2, slot = k == 0 ? 0 : 1;
    tot = wpart[iq][w0][slot];
    for (int w = w0 + step; w < kBlock / 64; w += step) tot = comp_merge(tot, wpart[iq][w][slot]);
  }
  if (S > 1) {
    // Hand the slice's sums over and take a ticket; the last slice merges them
    // all in slice order.  The slices run on several XCDs, whose L2s do not see
    // each other's lines: `part` and the ticket are read and written by
    // agent-scope atomics alone (never by plain accesses): on gfx950 those are
    // coherent over the XCDs (the loads and stores go past the L2s), and a wave's
    // s_waitcnt vmcnt(0) returns when its stores are done for all of them.  So
    // every sum stands before its ticket counts, and the loads behind the last
    // ticket, issued after its value came back, find them.  A release fence here
    // and an acquire fence there would also write back and invalidate the whole
    // L2, which nothing here needs: 64 transforms of 128 bins 33.6 -> 38.0 us a
    // call, 200 of 64 bins 48.7 -> 54.9.
    uint64_t* part = (uint64_t*)L.part + ((size_t)t * S * n_q * 3 + (size_t)lane) * 2;
    const size_t stride = (size_t)n_q * 6;  // words of a slice
    if (iq < n_q) {
      __hip_atomic_store(part + s * stride, (uint64_t)__double_as_longlong(tot.s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(part + s * stride + 1, (uint64_t)__double_as_longlong(tot.c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint32_t ticket = 0;
    if (lane == 0)
      ticket = (uint32_t)(__hip_atomic_fetch_add(&L.count[t], 1ull << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32);
    ticket = __builtin_amdgcn_readfirstlane(ticket);
    if (ticket != (uint32_t)S - 1) return;
    asm volatile("" ::: "memory");
    if (iq < n_q) {
      for (int j0 = 0; j0 < S; j0 += kLineLoads) {
        uint64_t v[kLineLoads][2];
#pragma unroll
        for (int j = 0; j < kLineLoads; ++j)
#pragma unroll
          for (int w = 0; w < 2; ++w)
            v[j][w] = j0 + j < S ? __hip_atomic_load(part + (j0 + j) * stride + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
#pragma unroll
        for (int j = 0; j < kLineLoads; ++j) {
          if (j0 + j >= S) break;
          const Comp o = {__longlong_as_double((int64_t)v[j][0]), __longlong_as_double((int64_t)v[j][1])};
          tot = j0 + j == 0 ? o : comp_merge(tot, o);
        }
      }
    }
    if (lane == 0) __hip_atomic_store(&L.count[t], (uint64_t)n_int, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const double sum = tot.s + tot.c;
  const int l3 = lane < n_q ? 3 * lane : 0;
  const double sj = __shfl(sum, l3, 64), sf = __shfl(sum, l3 + 1, 64), sm = __shfl(sum, l3 + 2, 64);
  if (lane == 0 && L.overlap_out) L.overlap_out[t] = n_int;
  if (lane >= n_q) return;
  const double q = L.q.q[lane], qm1 = q - 1.0;
  double I;
  if (q == 1.0) {
    I = (sj - sf) - sm;
  } else {
    const double Sj = -sj / qm1, Sf = -sf / qm1, Sm = -sm / qm1;
    I = (Sf + Sm) - Sj;
    if (L.q.pseudo) I += (1.0 - q) * Sf * Sm;
  }
  mi[lane] = I;
}

template <bool TABLE>
static void reduce_variant(const ReduceLaunch& L, unsigned blocks, hipStream_t s) {
  const int rows = (L.bins + L.splits - 1) / L.splits;
  if (rows * L.bins <= kBlock * kCellsFew)
    hipLaunchKernelGGL((mi_reduce_kernel<TABLE, kCellsFew>), dim3(blocks), dim3(kBlock), 0, s, L);
  else
    hipLaunchKernelGGL((mi_reduce_kernel<TABLE, kCellsMany>), dim3(blocks), dim3(kBlock), 0, s, L);
}

hipError_t launch_mi_reduce(const ReduceLaunch& Lin, hipStream_t s) {
  if (Lin.n == 0) return hipSuccess;
  ReduceLaunch L = Lin;
  L.splits = reduce_splits(L.bins, L.n);
  hipError_t e;
  const int S = L.splits;
  // launches of whole transforms, each below 2^31 work-items; the slice
  // count stays that of the whole batch
  const size_t BB = (size_t)L.bins * L.bins;
  const int32_t step = transforms_per_launch(S, kBlock);
  for (int32_t t0 = 0; t0 < L.n; t0 += step) {
    ReduceLaunch P = L;
    P.n = L.n - t0 < step ? L.n - t0 : step;
    if (L.hist) P.hist = L.hist + (size_t)t0 * BB;
    if (L.table) P.table = L.table + (size_t)t0 * BB;
    P.count = L.count + t0;
    P.part = L.part + (size_t)t0 * S * L.q.n * 3 * 2;  // (sum, error) pairs
    P.transforms = L.transforms + 12 * (size_t)t0;
    if (L.marg_out) P.marg_out = L.marg_out + (size_t)t0 * 2 * L.bins;
    P.mi_out = L.mi_out + (size_t)t0 * L.q.n;
    if (L.overlap_out) P.overlap_out = L.overlap_out + t0;
    const unsigned blocks = (unsigned)((int64_t)P.n * S);
    if (P.table)
      reduce_variant<true>(P, blocks, s);
    else
      reduce_variant<false>(P, blocks, s);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gemi
