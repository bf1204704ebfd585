// Pair form of the symmetric fine-level operator and its products (gfx950).
//
// The V-scaled matrix is symmetric (a_ij and a_ji are the same bits), so a
// product needs every pair once: y_i += a_ij x_j and y_j += a_ij x_i.  A
// product over the full rows is bound by the bytes of its entries; the pair
// form halves them.  Rows are cut into tiles of kTileRows.  A tile holds the
// pairs (i, j) of its rows i with j > i, and numbers the columns it meets
// locally: its own rows 0..255, then the columns of later tiles (its external
// columns, ascending, xcol[xoff[t] ...)).  Pairs are stored row by row in
// groups of four, the last group of a row filled up with zero values on
// one column past the tile's own, where x reads as zero and the sums are
// dropped (an infinite x elsewhere must not meet a zero value): one row byte,
// four 16-bit local columns and four values per group.  The 256 threads of a
// tile's block take equal runs of consecutive groups, and the groups are stored in the order of that walk (step k of
// thread T at 256 k + T): loads are contiguous over a wave, there are no row
// pointers and no ragged ends, a thread keeps its row's sum in a register, and
// the lanes of a wave hold different rows, so that their LDS adds seldom meet
// (with consecutive groups on consecutive lanes a row of 125 pairs put 32
// lanes on one address).  FP64 values are stored as two planes per tile
// (entries 0-1 of every group, then entries 2-3), so that each 16-byte load
// instruction reads one contiguous run.
//
// A product stages x of the tile's columns in LDS and adds both sides of
// every pair into FP64 LDS accumulators, one set per wave, so that the order
// of the additions is fixed.  The four sets are summed in wave order; sums of
// own rows go to y, sums of external columns to the tile's places in an
// exchange buffer.  The next kernel that reads y adds, for row j, the sums that
// earlier tiles left for it (pair_in), in ascending order of the tiles.
//
// Bound: HBM in FP64 (4.5 TB/s of entries at 2.1M Wendland rows, 602 us, and
// 4.4 TB/s at 16.8M cubic-spline rows, 1131 us), the LDS adds in FP32 (about
// one lane per clock and CU: 374 and 732 us).  ds_add_f32 runs at a third of the rate of ds_add_f64 here (2.8
// ms against 1.1 ms a product of 16.8M rows), so FP32 products add in FP64 as
// well.  Plain LDS reads and writes with one row per 32 lanes and a set per row
// need no atomics, but took 2.6 ms (FP64) and 1.27 ms (FP32).
#pragma once

#include "internal.h"
#include "reduce.h"
#include "spmv.h"

namespace rt {

// Sum of what earlier tiles left for row i (part: the exchange buffer).  A
// 3-D cubic-spline row has two such sums on average, at most about ten: four
// places, then four sums are requested at a time.
template <typename T>
__device__ __forceinline__ T pair_in(const PairIn& P, int64_t i, const T* __restrict__ part) {
  const int k0 = P.ptr[i], k1 = P.ptr[i + 1];
  T s = 0;
  for (int k = k0; k < k1; k += 4) {
    int at[4];
    T v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = k + q < k1 ? P.pos[k + q] : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = at[q] >= 0 ? part[at[q]] : T(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) s += v[q];
  }
  return s;
}

// what a pair product forms beside the exchange sums
enum PairMode {
  PP_DOT = 0,   // y = own part of A x, part[block] = this tile's share of x.A x
  PP_PLAIN = 1, // y = own part of A x
  PP_ONES = 2   // y = own part of (A - diag) 1 (x and diag not read)
};

template <typename T> struct PairLoad;
template <> struct PairLoad<float> {
  rt_f32x4 v;
  __device__ __forceinline__ void load(const float* val, int g, int) {
    v = stream_load(reinterpret_cast<const rt_f32x4*>(val) + g);
  }
  __device__ __forceinline__ float at(int q) const { return v[q]; }
};
template <> struct PairLoad<double> {
  rt_f64x2 a, b;
  __device__ __forceinline__ void load(const double* val, int g, int ng) {
    a = stream_load(reinterpret_cast<const rt_f64x2*>(val) + g);
    b = stream_load(reinterpret_cast<const rt_f64x2*>(val) + ng + g);
  }
  __device__ __forceinline__ double at(int q) const { return q < 2 ? a[q] : b[q - 2]; }
};

constexpr int kPairSets = kBlock / kWave;   // accumulator sets of a product

// LDS bytes of a product over tiles of at most ncol columns
template <typename T>
inline size_t pair_lds(int ncol) {
  return (sizeof(double) * kPairSets + sizeof(T)) * (size_t)(ncol + 1);
}

// U groups of a thread: steps k .. k + U - 1 of its run.  The loads are not
// predicated (past the end they read the tile's last group again, which add()
// leaves out; an empty tile reads the first group after its own): behind a
// branch the compiler cannot count the loads in flight and waits for all of
// them, those just issued included.
template <typename T, int U>
struct PairBatch {
  PairLoad<T> v[U];
  rt_u16x4 c[U];
  int r[U];
  __device__ __forceinline__ void load(const T* vt, const rt_u16x4* ct, const uint8_t* rows, int k,
                                       int ng) {
    const int last = max(ng - 1, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = min((k + u) * kBlock + (int)threadIdx.x, last);
      v[u].load(vt, g, ng);
      c[u] = stream_load(ct + g);
      r[u] = stream_load(rows + g);
    }
  }
  // cur: the row whose sum s is, xr its x
  template <int MODE>
  __device__ __forceinline__ void add(const T* xs, double* mine, int ncol, int k, int ng, int& cur,
                                      T& xr, T& s) const {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = (k + u) * kBlock + (int)threadIdx.x < ng;
      const bool turn = in && r[u] != cur;
      RT_WAVE_LDS_ADD(turn && cur >= 0, mine + cur, (double)s);
      if (turn) {
        cur = r[u];
        s = 0;
        if (MODE != PP_ONES) xr = xs[cur];
      }
      if (in) {
#pragma unroll
        for (int q = 0; q < 4; ++q) s += MODE == PP_ONES ? v[u].at(q) : v[u].at(q) * xs[c[u][q]];
      }
      // The filling's sums are dropped; on short rows (U = 1), where it is a tenth of
      // the entries and meets in one address, they are not formed either (1% of a
      // step of 1M particles of 36 neighbours; on rows of 255 the test costs 1%).
#pragma unroll
      for (int q = 0; q < 4; ++q)
        RT_WAVE_LDS_ADD(in && (U > 1 || q == 0 || c[u][q] < ncol), mine + c[u][q],
                        (double)v[u].at(q) * (double)xr);
    }
  }
};

template <typename T, int U, int MODE>
__global__ void __launch_bounds__(kBlock)
k_pair_spmv(int64_t n, int per, int64_t ntiles, PairArgs A, const T* __restrict__ val,
            const T* __restrict__ diag, const T* __restrict__ x, T* __restrict__ y,
            T* __restrict__ xsum, double* __restrict__ part, const int32_t* __restrict__ tprob,
            const int32_t* __restrict__ skip) {
  RT_DYNAMIC_LDS(dyn_lds);
  __shared__ double red[kBlock / kWave];
  const int t = xcd_block(per, tprob != nullptr);
  const int tid = threadIdx.x;
  if (t >= ntiles) {   // grids are padded to a multiple of the XCD count
    if (MODE == PP_DOT && tid == 0 && part) part[t] = 0.0;
    return;
  }
  if (skip && skip[tprob ? tprob[t] : 0]) return;   // a finished problem's tile
  const int64_t r0 = (int64_t)t * kTileRows;
  const int64_t i = r0 + tid;
  const bool live = i < n;
  const int64_t x0 = A.xoff[t];
  const int next = (int)(A.xoff[t + 1] - x0);
  const int ncol = kTileRows + next;
  const int64_t g0 = A.goff[t];
  const int ng = A.gcnt[t];
  const T* vt = val + 4 * g0;
  const rt_u16x4* ct = reinterpret_cast<const rt_u16x4*>(A.col + 4 * g0);
  const uint8_t* rows = A.row + g0;
  const int nset = ncol + 1;   // and the filling's column (8 or 32 of them: 0.6% of a 16.8M step)
  double* acc = reinterpret_cast<double*>(dyn_lds);   // kPairSets sets of nset
  T* xs = reinterpret_cast<T*>(acc + kPairSets * nset);
  PairBatch<T, U> b0, b1;
  b0.load(vt, ct, rows, 0, ng);   // in flight while the columns are staged
  T di = 0;
  if (MODE != PP_ONES) {
    if (live) di = diag[i];
    xs[tid] = live ? x[i] : T(0);
    for (int k = tid; k < next; k += kBlock) xs[kTileRows + k] = x[A.xcol[x0 + k]];
    if (tid == 0) xs[ncol] = T(0);
  }
  for (int k = tid; k < kPairSets * nset; k += kBlock) acc[k] = 0.0;
  __syncthreads();
  double* mine = acc + (tid / kWave) * nset;
  T s = 0, xr = 1;
  int cur = -1;
  for (int k = 0; k * kBlock < ng; k += 2 * U) {
    b1.load(vt, ct, rows, k + U, ng);
    b0.template add<MODE>(xs, mine, ncol, k, ng, cur, xr, s);
    b0.load(vt, ct, rows, k + 2 * U, ng);
    b1.template add<MODE>(xs, mine, ncol, k + U, ng, cur, xr, s);
  }
  RT_WAVE_LDS_ADD(cur >= 0, mine + cur, (double)s);
  __syncthreads();
  double dot = 0.0;
  {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kPairSets; ++w) sum += acc[w * nset + tid];
    if (MODE != PP_ONES) sum = (double)di * (double)xs[tid] + sum;
    if (live) {
      y[i] = (T)sum;
      if (MODE == PP_DOT) dot = (double)xs[tid] * sum;
    }
  }
  for (int k = kTileRows + tid; k < ncol; k += kBlock) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kPairSets; ++w) sum += acc[w * nset + k];
    xsum[x0 + k - kTileRows] = (T)sum;
    if (MODE == PP_DOT) dot += (double)xs[k] * sum;
  }
  if (MODE == PP_DOT) {
    dot = block_sum(dot, red);
    if (tid == 0 && part) part[t] = dot;
  }
}

template <typename T> struct PairSel;
template <> struct PairSel<double> {
  static const double* val(const PairForm& P) { return P.val64.p; }
  static double* sum(const PairForm& P) { return P.sum64.p; }
};
template <> struct PairSel<float> {
  static const float* val(const PairForm& P) { return P.val32.p; }
  static float* sum(const PairForm& P) { return P.sum32.p; }
};

// The pair form serves a product with the given shape request: the default
// and every tiled shape, whose rows in flight (1, 2 or 4) become groups in flight per
// thread; plain shapes run on the CSR rows where those are current.
inline bool plain_shape(int shape) {
  return shape >= 0 && shape < kNumSpmvShapes && !kSpmvShapes[shape].tiled;
}
// whether a solve that multiplies with this shape needs the CSR rows made
inline bool wants_rows(const Level& L, int shape) {
  return L.pair.on && (plain_shape(shape) || plain_shape(resid_shape(L)));
}
inline bool pair_serves(const Level& L, int shape) {
  return L.pair.on && (!plain_shape(shape) || !L.csr_vals);
}
// Groups in work per thread without a request (as many again are loading): two,
// one where rows are so short (a thread takes about row/8 groups) that a run
// ends before wider batches pay.  Measured per product, 1 / 2 / 4 groups: FP64
// 698 / 602 / 604 us and FP32 424 / 374 / 362 us at 2.1M Wendland rows (255
// neighbours), FP64 1136 / 1131 / 1160 us and FP32 754 / 732 / 756 us at 16.8M
// cubic-spline rows (57), FP64 14.8 / 15.7 / 18.2 us and FP32 14.0 / 14.3 /
// 16.1 us at 262k rows of 38.
inline int pair_groups(const Level& L) { return L.nnz >= 50 * L.n ? 2 : 1; }

// Own part of A x over the level into y and the exchange sums into the
// level's buffer (PairMode); *nparts receives the partials written (PP_DOT).
template <typename T, int MODE>
int launch_pair(hipStream_t st, const Level& L, const T* diag, const T* x, T* y, double* part,
                int* nparts, int shape = -1, const int32_t* tprob = nullptr,
                const int32_t* skip = nullptr) {
  const PairForm& P = L.pair;
  const int grid = spmv_blocks_rows(L.n, kTileRows, tprob != nullptr);
  const int per = grid / kXcd;
  if (nparts) *nparts = grid;
  if (L.n == 0) return RT_OK;
  const int u = shape >= 0 && shape < kNumSpmvShapes ? kSpmvShapes[shape].ent : pair_groups(L);
  const size_t lds = pair_lds<T>(kTileRows + P.max_ext);
#define RT_PAIR_U(U_)                                                                            \
  hipLaunchKernelGGL((k_pair_spmv<T, U_, MODE>), dim3(grid), dim3(kBlock), lds, st, L.n, per,     \
                     P.ntiles, P.args(), PairSel<T>::val(P), diag, x, y, PairSel<T>::sum(P), part, \
                     tprob, skip)
  if (u == 1) RT_PAIR_U(1);
  else if (u == 2) RT_PAIR_U(2);
  else RT_PAIR_U(4);
#undef RT_PAIR_U
  RT_LAUNCH_CHECK();
  return RT_OK;
}

}  // namespace rt
