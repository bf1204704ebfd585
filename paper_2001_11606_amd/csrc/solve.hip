// Preconditioned conjugate gradients for the V-scaled radiation system
// (the D^-1 operator of Sec. 3.2), FP64 and mixed precision.
//
// The paper solves the diffusion equation with AMG-preconditioned GMRES; the
// V-scaled matrix here is symmetric positive definite, so CG applies.  The
// paper warm-starts with E^l; the caller passes the initial guess in x.
//
// FP64:  PCG on A x = b, stop when ||r||_2 <= tol ||b||_2 (recursive residual).
// MIXED: r = b - A x in FP64; repeat { FP32 PCG on A d = r (FP32 matrix, FP32
//        vectors and arithmetic) to a relative reduction inner_tol (or just
//        enough to reach tol); x += d in FP64; r = b - A x in FP64 } until
//        ||r||_2 <= tol ||b||_2 -- the classical iterative refinement.
// Componentwise test (cw_tol > 0): both precisions also require
// max_i |r_i| / (a_ii |x_i|) <= cw_tol, the largest relative change of one
// unknown that a Jacobi sweep would still make.  A normwise test alone is
// blind to unknowns many decades below the largest: on a radiation front E
// spans eight decades, and rows near 1e-8 can keep relative errors of 1e-9
// under ||r|| <= 1e-14 ||b||.  The FP32 inner solve then measures its
// residual with the weights 1/(a_ii |x_i|) of the refinement's start.
//
// Scalars (alpha, beta, r.z, ...) and thresholds stay on the device; block
// partials of the dot products are combined in FP64 in a fixed order.  Up to
// a few thousand of them, every block of the kernel that needs a scalar
// combines them itself (all get the same bits, block 0 keeps the record);
// beyond that a one-block kernel does.  An iteration is then three launches
// instead of five: below 1M rows the one-block kernels took 5.5 us each, as
// long as a vector pass.
// The stopping test runs on the device too: the residual's first reduction
// (k_start) sets the thresholds and a stop flag, the kernel that forms ||r||^2
// sets the flag once the threshold is met (or on breakdown), and every kernel
// of the iteration does nothing once it is set.  The flag is kept in two words
// (STOP_X, STOP_P), so that no launch reads the word it writes: the waves of a
// block read it one by one, and those that went on while the others left would
// combine sums with shares missing.  The host queues the start and
// several iterations between reads of the state -- as many as the observed
// convergence rate says are still needed, scaled down so that it rarely
// queues past the end -- so neither a start nor an iteration costs a host
// round trip, and the arithmetic is the same as stopping after each iteration.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "internal.h"
#include "pair.h"
#include "reduce.h"
#include "spmv.h"

namespace rt {
namespace {

// device scalars; S_RZ holds r.z in two places that the iterations alternate
// between (a kernel whose blocks read one writes the other)
enum { S_RZ = 0, S_RZ_ALT, S_PQ, S_ALPHA, S_BETA, S_RR, S_RR0, S_CW0, S_BB, S_BAD, S_ITS, S_STOP,
       S_CW, S_RZ_PREV, S_RZ_LAST, S_THR, S_CWTHR, S_DONE, S_MIS, S_COUNT };
// The two words of the stop flag.  The product and the x, r update read STOP_X;
// the preconditioner and the p update read STOP_P.  The x, r update sets STOP_P
// (breakdown, or STOP_X is set), the p update STOP_X (the loop ends, or STOP_P is
// set); the one-block kernels between launches set both.
enum { STOP_X = 0, STOP_P = 1, STOP_WORDS };
// componentwise measure of the update kernel: none, |r_i| w_i / |x_i| with
// w = 1/diag (the iterate's own measure), or |r_i| w_i with fixed weights
enum { CW_NONE = 0, CW_X = 1, CW_W = 2 };
enum { FIN_ALPHA = 0, FIN_BETA, FIN_RZ, FIN_RR, FIN_BB, FIN_RESUME };
enum { PROF_SPMV64 = 0, PROF_SPMV32 = 1, PROF_RESID64 = 2, PROF_KINDS = 3 };

// Sums of up to np partials in every block that calls it, and the largest of
// pc (pb, pc: NULL, none).  Four independent running sums per thread keep
// four loads in flight; they are combined in a fixed order.
struct Combined {
  double a, b, c;
};
__device__ __forceinline__ Combined combine(int np, const double* __restrict__ pa,
                                            const double* __restrict__ pb,
                                            const double* __restrict__ pc, double* red) {
  __shared__ Combined out;
  double c = 0.0;
  if (pc) {
    for (int k = threadIdx.x; k < np; k += kBlock) c = fmax(c, pc[k]);
    c = block_max(c, red);
  }
  double a4[4] = {0.0, 0.0, 0.0, 0.0}, b4[4] = {0.0, 0.0, 0.0, 0.0};
  int i = threadIdx.x;
  for (; i + 3 * kBlock < np; i += 4 * kBlock) {
#pragma unroll
    for (int u = 0; u < 4; ++u) a4[u] += pa[i + u * kBlock];
    if (pb) {
#pragma unroll
      for (int u = 0; u < 4; ++u) b4[u] += pb[i + u * kBlock];
    }
  }
  for (int u = 0; i < np; i += kBlock, ++u) {
    a4[u] += pa[i];
    if (pb) b4[u] += pb[i];
  }
  double a = block_sum((a4[0] + a4[1]) + (a4[2] + a4[3]), red);
  double b = 0.0;
  if (pb) b = block_sum((b4[0] + b4[1]) + (b4[2] + b4[3]), red);
  if (threadIdx.x == 0) out = Combined{a, b, c};
  __syncthreads();
  return out;
}

// alpha = r.z / p.Ap for the iteration that reads r.z from s[S_RZ + slot];
// returns false (and the record, by the calling block's thread 0 if keep, sets
// *word) on breakdown: p.Ap not positive
__device__ __forceinline__ bool take_alpha(double pq, int slot, double* __restrict__ s,
                                           int32_t* __restrict__ word, bool keep, double* alpha) {
  const bool ok = pq > 0.0 && isfinite(pq);
  *alpha = ok ? s[S_RZ + slot] / pq : 0.0;
  if (keep && threadIdx.x == 0) {
    s[S_PQ] = pq;
    s[S_ALPHA] = *alpha;
    if (!ok) {
      s[S_BAD] = 1.0;
      s[S_STOP] = 1.0;
      *word = 1;
    }
  }
  return ok;
}

// beta of the iteration from rr = ||r||^2, rz = r.z (new) and the componentwise
// measure cw (tested if has_cw); returns false (and sets *word) when the loop
// ends here
__device__ __forceinline__ bool take_beta(double rr, double rz, double cw, bool has_cw, int slot,
                                          double* __restrict__ s, int32_t* __restrict__ word,
                                          bool keep, double* beta) {
  const double last = s[S_RZ + slot];
  const bool ends = !(rr > s[S_THR]) && (!has_cw || !(cw > s[S_CWTHR]));
  *beta = rz / last;
  if (keep && threadIdx.x == 0) {
    s[S_RR] = rr;
    s[S_BETA] = *beta;
    s[S_RZ_PREV] = last;
    s[S_RZ_LAST] = rz;
    s[S_RZ + (slot ^ 1)] = rz;
    s[S_ITS] += 1.0;
    if (has_cw) s[S_CW] = cw;
    if (ends) {
      s[S_STOP] = 1.0;
      *word = 1;
    }
  }
  return !ends;
}

// One block: combine the partials and update the scalars; nothing happens
// once the stop flag is set, except for the norms (FIN_RR, FIN_BB).  Every wave
// has read the flag before thread 0, behind the barriers of combine, sets it.
__global__ void __launch_bounds__(kBlock)
k_finalize(int op, int np, const double* __restrict__ pa, const double* __restrict__ pb,
           const double* __restrict__ pc, double* __restrict__ s, int32_t* __restrict__ stop,
           int slot) {
  __shared__ double red[kBlock / kWave];
  if (op != FIN_RR && op != FIN_BB && stop[op == FIN_BETA ? STOP_P : STOP_X]) return;
  const Combined v = combine(np, pa, pb, pc, red);
  double unused;
  switch (op) {
    case FIN_ALPHA:
      if (!take_alpha(v.a, slot, s, stop + STOP_X, true, &unused) && threadIdx.x == 0)
        stop[STOP_P] = 1;
      break;
    case FIN_BETA:
      if (!take_beta(v.a, v.b, v.c, pc != nullptr, slot, s, stop + STOP_X, true, &unused) &&
          threadIdx.x == 0)
        stop[STOP_P] = 1;
      break;
    default:
      if (threadIdx.x != 0) return;
      if (op == FIN_RZ) {   // r.z at the start
        s[S_RZ] = v.a;
      } else if (op == FIN_RR) {
        s[S_RR] = v.a;
        if (pc) s[S_CW] = v.c;
      } else if (op == FIN_BB) {
        s[S_BB] = v.a;
      } else {   // FIN_RESUME: r.z of a residual that replaced the recursive one
        // The loop that stopped kept its last search direction and, in
        // S_RZ_PREV, the r.z it was formed with: beta continues from it, but
        // only while the replacement agrees with the recursion (S_RZ_LAST, the
        // recursive r.z it stopped at, within 25%).  The FP32 operator's own
        // error can make the two differ by far more than rounding; then
        // beta = 0, a restart (p = z).
        s[S_BETA] = s[S_RZ_PREV] > 0.0 && isfinite(s[S_RZ_PREV]) && v.a >= 0.75 * s[S_RZ_LAST] &&
                            v.a <= 1.25 * s[S_RZ_LAST]
                        ? v.a / s[S_RZ_PREV]
                        : 0.0;
        s[S_RZ] = v.a;
      }
  }
}

// Thresholds of a solve and of its inner loop.
struct Tolerances {
  double tol2, cwthr;    // ||r||^2 <= tol2 ||b||^2 and the componentwise measure <= cwthr
  double inner_tol;      // MIXED: reduction asked of the inner loop; 0: FP64
};

// One block, before an inner loop: the residual's norm and componentwise
// measure (pr, pc), with pb also ||b||^2; whether the solve is done, else the
// inner loop's thresholds.  *mismatch (else NULL) non-zero: the residual is
// not that of the caller's state, nothing runs on it.
__global__ void __launch_bounds__(kBlock)
k_start(int npr, const double* __restrict__ pr, const double* __restrict__ pc, int npb,
        const double* __restrict__ pb, const int32_t* __restrict__ mismatch, Tolerances t,
        double* __restrict__ s, int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  const Combined v = combine(npr, pr, nullptr, pc, red);
  __syncthreads();
  double bb = 0.0;
  if (pb) bb = combine(npb, pb, nullptr, nullptr, red).a;
  if (threadIdx.x != 0) return;
  if (pb) s[S_BB] = bb;
  else bb = s[S_BB];
  const double rr = v.a, cw = v.c, thr2 = t.tol2 * bb;
  const bool mis = mismatch && *mismatch != 0;
  // (a residual that is not a number ends refinements, not the FP64 loop)
  const bool done = (t.inner_tol > 0.0 ? !(rr > thr2) : rr <= thr2) && !(cw > t.cwthr);
  s[S_RR] = s[S_RR0] = rr;
  s[S_CW] = s[S_CW0] = cw;
  s[S_MIS] = mis ? 1.0 : 0.0;
  s[S_DONE] = done ? 1.0 : 0.0;
  if (t.inner_tol > 0.0) {
    // reduce by inner_tol, or just enough (with margin) to reach the
    // tolerance; the same for the componentwise measure when it is tested
    const double f = fmax(t.inner_tol, 0.3 * sqrt(thr2 / rr));
    s[S_THR] = f * f * rr;
    s[S_CWTHR] = t.cwthr < INFINITY ? fmax(t.inner_tol, 0.3 * t.cwthr / cw) * cw : INFINITY;
  } else {
    s[S_THR] = thr2;
    s[S_CWTHR] = t.cwthr;
  }
  const bool halt = mis || done || bb == 0.0 || !isfinite(bb);
  s[S_BAD] = 0.0;
  s[S_ITS] = 0.0;
  s[S_STOP] = halt ? 1.0 : 0.0;
  stop[STOP_X] = stop[STOP_P] = halt ? 1 : 0;
}

// Streaming vector kernels: kVec elements per thread (coalesced per element
// slot), one up to kVecOne rows, where four leave most of the chip idle; one
// partial per block, no grid-stride loop.  Beyond, the partials that every
// block combines cost more than the idle units: steps with one | four elements
// of 27k rows 550 | 600 us, 512k 6.8 | 6.3 ms, 1M 12.7 | 10.3 ms; at 262k
// 1.32 | 1.35 ms (FP64, 255 neighbours) and 4.20 | 4.15 ms (FP32, 38).
constexpr int kVec = 4;
constexpr int64_t kVecOne = (int64_t)1 << 17;
__host__ __device__ inline int vec_per_thread(int64_t n) { return n <= kVecOne ? 1 : kVec; }
inline int vec_blocks(int64_t n) {
  const int64_t per_block = (int64_t)kBlock * vec_per_thread(n);
  return (int)std::max<int64_t>(1, (n + per_block - 1) / per_block);
}
#define RT_VEC_LOOP(i)                                                                  \
  for (int _u = 0, _e = vec_per_thread(n); _u < _e; ++_u)                               \
    for (int64_t i = ((int64_t)blockIdx.x * _e + _u) * kBlock + threadIdx.x; i < n; i = n)

// second reduction level: nb2 blocks each sum a contiguous chunk of pa (and pb)
__global__ void __launch_bounds__(kBlock)
k_partial_reduce(int np, int chunk, const double* __restrict__ pa, const double* __restrict__ pb,
                 const double* __restrict__ pc, double* __restrict__ out,
                 const int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  if (stop && *stop) return;
  const int lo = blockIdx.x * chunk;
  const int hi = lo + chunk < np ? lo + chunk : np;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int i = lo + threadIdx.x; i < hi; i += kBlock) {
    a += pa[i];
    if (pb) b += pb[i];
    if (pc) c = fmax(c, pc[i]);
  }
  a = block_sum(a, red);
  b = block_sum(b, red);
  if (pc) c = block_max(c, red);
  if (threadIdx.x == 0) {
    out[blockIdx.x] = a;
    out[gridDim.x + blockIdx.x] = b;
    out[2 * gridDim.x + blockIdx.x] = c;
  }
}

// p = M r for Jacobi (M = diag^-1), part = r.p
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_init_jacobi(int64_t n, const T* __restrict__ dinv, const T* __restrict__ r, T* __restrict__ p,
              double* __restrict__ part, const int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  if (*stop) return;
  double acc = 0.0;
  RT_VEC_LOOP(i) {
    const T z = dinv[i] * r[i];
    p[i] = z;
    acc += (double)r[i] * (double)z;
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// part = r.(D^-1 r): the r.z of a Jacobi-preconditioned residual
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_rz_jacobi(int64_t n, const T* __restrict__ dinv, const T* __restrict__ r,
            double* __restrict__ part, const int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  if (*stop) return;
  double acc = 0.0;
  RT_VEC_LOOP(i) acc += (double)r[i] * (double)(dinv[i] * r[i]);
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// p = z, part = r.z
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_copy_dot(int64_t n, const T* __restrict__ r, const T* __restrict__ z, T* __restrict__ p,
           double* __restrict__ part, const int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  if (*stop) return;
  double acc = 0.0;
  RT_VEC_LOOP(i) {
    p[i] = z[i];
    acc += (double)r[i] * (double)z[i];
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

template <typename T>
__global__ void __launch_bounds__(kBlock)
k_dot(int64_t n, const T* __restrict__ a, const T* __restrict__ b, double* __restrict__ part,
      const int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  if (stop && *stop) return;
  double acc = 0.0;
  RT_VEC_LOOP(i) acc += (double)a[i] * (double)b[i];
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// x += alpha p; r -= alpha q; partA = r.r; (Jacobi) partB = r.(dinv r);
// CW != CW_NONE: partC = the block maximum of the componentwise measure, with
// w = dinv (CW_X: |r_i| w_i / |x_i| of the updated x) or fixed weights (CW_W)
// PAIR: q holds each tile's own part of A p, completed here (pair_in)
// npq > 0: alpha is formed here from the product's npq partials (block 0
// keeps the record), else it is s[S_ALPHA].
// The first element's loads, which do not wait for alpha, are in flight while
// the partials are combined (16.4k FP64 rows, one element per thread: 9.7 ->
// 5.5 us; steps of 1M rows, four: 10.12 -> 10.04 ms).  Those of all four would
// cost registers and with them waves (FP32, 16.8M rows: 109 -> 138 us).
template <typename T, bool JAC, int CW, bool PAIR, int E>
__global__ void __launch_bounds__(kBlock)
k_update(int64_t n, PairIn P, const T* __restrict__ qsum, int npq, const double* __restrict__ pq,
         int slot, double* __restrict__ s, T* __restrict__ x, T* __restrict__ r,
         const T* __restrict__ p, const T* __restrict__ q, const T* __restrict__ dinv,
         const T* __restrict__ w, double* __restrict__ partA, double* __restrict__ partB,
         double* __restrict__ partC, int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  const bool keep = blockIdx.x == 0;
  if (stop[STOP_X]) {   // read by this launch, never written by it
    if (keep && threadIdx.x == 0) stop[STOP_P] = 1;
    return;
  }
  struct Row {
    T x, p, q, r, dinv, w;
  };
  auto load = [&](int64_t i) {
    Row v;
    v.x = x[i];
    v.p = p[i];
    v.q = q[i];
    v.r = r[i];
    v.dinv = JAC ? dinv[i] : T(0);
    v.w = CW != CW_NONE ? w[i] : T(0);
    if (PAIR) v.q += pair_in<T>(P, i, qsum);
    return v;
  };
  const int64_t i0 = (int64_t)blockIdx.x * kBlock * E + threadIdx.x;
  Row first{};
  if (i0 < n) first = load(i0);
  double al = 0.0;
  if (npq > 0) {
    const Combined v = combine(npq, pq, nullptr, nullptr, red);
    if (!take_alpha(v.a, slot, s, stop + STOP_P, keep, &al)) return;
  } else {
    al = s[S_ALPHA];
  }
  const T alpha = (T)al;
  double rr = 0.0, rz = 0.0, cw = 0.0;
  for (int e = 0; e < E; ++e) {
    const int64_t i = i0 + e * kBlock;
    if (i >= n) break;
    const Row v = e == 0 ? first : load(i);
    const T xi = v.x + alpha * v.p;
    x[i] = xi;
    const T ri = v.r - alpha * v.q;
    r[i] = ri;
    rr += (double)ri * (double)ri;
    if (JAC) rz += (double)ri * (double)(v.dinv * ri);
    if (CW == CW_X) {
      const double ax = fabs((double)xi);
      const double t = fabs((double)ri) * (double)v.w;
      cw = fmax(cw, ax > 0.0 ? t / ax : (ri == T(0) ? 0.0 : INFINITY));
    } else if (CW == CW_W) {
      cw = fmax(cw, fabs((double)ri) * (double)v.w);
    }
  }
  rr = block_sum(rr, red);
  if (JAC) rz = block_sum(rz, red);
  if (CW != CW_NONE) cw = block_max(cw, red);
  if (threadIdx.x == 0) {
    partA[blockIdx.x] = rr;
    if (JAC) partB[blockIdx.x] = rz;
    if (CW != CW_NONE) partC[blockIdx.x] = cw;
  }
}

// p = z + beta p, with z = dinv r (Jacobi) or the preconditioned vector
// np > 0: beta is formed here from the np partials of r.r, r.z and, with pc,
// the componentwise measure (block 0 keeps the record), else it is s[S_BETA]
template <typename T, bool JAC, int E>
__global__ void __launch_bounds__(kBlock)
k_pupdate(int64_t n, int np, const double* __restrict__ pa, const double* __restrict__ pb,
          const double* __restrict__ pc, int slot, double* __restrict__ s,
          const T* __restrict__ r, const T* __restrict__ dinv, const T* __restrict__ z,
          T* __restrict__ p, int32_t* __restrict__ stop) {
  __shared__ double red[kBlock / kWave];
  const bool keep = blockIdx.x == 0;
  if (stop[STOP_P]) {   // read by this launch, never written by it
    if (keep && threadIdx.x == 0) stop[STOP_X] = 1;
    return;
  }
  const int64_t i0 = (int64_t)blockIdx.x * kBlock * E + threadIdx.x;
  T zv[E], dv[E], pv[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {   // in flight while the partials are combined
    const int64_t i = i0 + e * kBlock < n ? i0 + e * kBlock : n - 1;
    zv[e] = JAC ? r[i] : z[i];
    dv[e] = JAC ? dinv[i] : T(1);
    pv[e] = p[i];
  }
  double be = 0.0;
  if (np > 0) {
    const Combined v = combine(np, pa, pb, pc, red);
    if (!take_beta(v.a, v.b, v.c, pc != nullptr, slot, s, stop + STOP_X, keep, &be)) return;
  } else {
    be = s[S_BETA];
  }
  const T beta = (T)be;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (i0 + e * kBlock >= n) break;
    p[i0 + e * kBlock] = (JAC ? dv[e] * zv[e] : zv[e]) + beta * pv[e];
  }
}

// Initial residual from the previous one: for the same matrix and x, b - A x =
// (b_prev - A x) + (b - b_prev).  r = r + (b - b_prev) (r32: its FP32 copy),
// partA = r.r, partB = b.b, partC = the block maximum of the componentwise
// measure |r_i| / (a_ii |x_i|) (x, diag), w32 (else NULL) its weights.
__global__ void __launch_bounds__(kBlock)
k_resid_shift(int64_t n, const double* __restrict__ b, const double* __restrict__ b_prev,
              const double* __restrict__ x, const double* __restrict__ diag,
              double* __restrict__ r, float* __restrict__ r32, float* __restrict__ w32,
              double* __restrict__ partA, double* __restrict__ partB,
              double* __restrict__ partC) {
  __shared__ double red[kBlock / kWave];
  double rr = 0.0, bb = 0.0, cw = 0.0;
  RT_VEC_LOOP(i) {
    const double bi = b[i];
    const double ri = r[i] + (bi - b_prev[i]);
    r[i] = ri;
    if (r32) r32[i] = (float)ri;
    rr += ri * ri;
    bb += bi * bi;
    const double xi = x[i], di = diag[i];
    cw = fmax(cw, cw_term(ri, di, xi));
    if (w32) w32[i] = cw_weight(di, xi);
  }
  rr = block_sum(rr, red);
  bb = block_sum(bb, red);
  cw = block_max(cw, red);
  if (threadIdx.x == 0) {
    partA[blockIdx.x] = rr;
    partB[blockIdx.x] = bb;
    partC[blockIdx.x] = cw;
  }
}

// x += d, d = 0 for the next inner loop
__global__ void k_add_f32(int64_t n, float* __restrict__ d, double* __restrict__ x) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) {
    x[i] += (double)d[i];
    d[i] = 0.f;
  }
}

template <typename T>
__global__ void k_zero(int64_t n, T* __restrict__ x) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0;
}

__global__ void k_gather(int64_t n, const int32_t* __restrict__ perm, const double* __restrict__ in,
                         double* __restrict__ out) {
  int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (s < n) out[s] = in[perm[s]];
}

__global__ void k_scatter(int64_t n, const int32_t* __restrict__ perm,
                          const double* __restrict__ in, double* __restrict__ out) {
  int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (s < n) out[perm[s]] = in[s];
}

struct Prof {
  rt_ctx* ctx;
  int kind;
  size_t a = 0;
  Prof(rt_ctx* c, int k) : ctx(c), kind(k) {}
  int begin() { return ctx->profiling ? ctx->prof_mark(&a) : RT_OK; }
  int end() {
    if (!ctx->profiling) return RT_OK;
    size_t b;
    RT_CHECK(ctx->prof_mark(&b));
    ctx->prof_spans.push_back({kind, a, b});
    return RT_OK;
  }
};

// Device buffers of one solve: work vectors of the fine level (n entries
// each; the FP32 ones only for mixed precision), block partials, the Krylov
// scalars and the stop flag.
struct Work {
  double *r64 = nullptr, *p64 = nullptr, *q64 = nullptr, *z64 = nullptr;
  float *r32 = nullptr, *p32 = nullptr, *q32 = nullptr, *z32 = nullptr, *d32 = nullptr,
        *w32 = nullptr;
  double *partA = nullptr, *partB = nullptr, *partC = nullptr, *partD = nullptr, *partF = nullptr,
         *scal = nullptr;
  int32_t* stop = nullptr;   // STOP_WORDS words
};

template <typename T> struct Sel;
template <> struct Sel<double> {
  static const double* val(const Level& L) { return L.val64.p; }
  static const double* diag(const Level& L) { return L.diag64.p; }
  static const double* dinv(const Level& L) { return L.dinv64.p; }
  static double* p(const Work& W) { return W.p64; }
  static double* q(const Work& W) { return W.q64; }
  static double* z(const Work& W) { return W.z64; }
  static constexpr int kind = PROF_SPMV64;
};
template <> struct Sel<float> {
  static const float* val(const Level& L) { return L.val32.p; }
  static const float* diag(const Level& L) { return L.diag32.p; }
  static const float* dinv(const Level& L) { return L.dinv32.p; }
  static float* p(const Work& W) { return W.p32; }
  static float* q(const Work& W) { return W.q32; }
  static float* z(const Work& W) { return W.z32; }
  static constexpr int kind = PROF_SPMV32;
};

// partial counts above which a second reduction level runs first
#ifndef RT_PARTIAL_FOLD_MIN
#define RT_PARTIAL_FOLD_MIN (4 * kMaxPartials)
#endif

// Partials a kernel's blocks combine themselves: of a product (one array, 32 KB
// read by every block) and of a vector pass (three arrays).  40 CG steps in FP64,
// combined by every block | by a launch of their own: product partials, 3456
// 3.75 | 3.82 ms, 4025 4.17 | 4.23, 5488 5.42 | 5.45, 8192 7.55 | 7.54; vector
// partials, 1372 5.46 | 5.52 ms, 1688 6.47 | 6.39, 2048 7.54 | 7.46, 2680 9.86 |
// 9.68, 4000 14.8 | 14.2 (FP32: 1688 4.98 | 5.02, 2680 7.41 | 7.34).
#ifndef RT_FUSED_PARTIALS
#define RT_FUSED_PARTIALS 4096
#endif
constexpr int kFusedVec = RT_FUSED_PARTIALS < 1536 ? RT_FUSED_PARTIALS : 1536;

// np partials folded to at most kMaxPartials when they are many
struct Partials {
  int np;
  const double *a, *b, *c;
};
int fold(rt_ctx* ctx, const Work& W, Partials* p, double* out, const int32_t* stop) {
  if (p->np <= RT_PARTIAL_FOLD_MIN) return RT_OK;
  const int nb2 = std::min(kMaxPartials, std::max(1, p->np / 8));
  const int chunk = (p->np + nb2 - 1) / nb2;
  hipLaunchKernelGGL(k_partial_reduce, dim3(nb2), dim3(kBlock), 0, ctx->stream, p->np, chunk, p->a,
                     p->b, p->c, out, stop);
  RT_LAUNCH_CHECK();
  *p = Partials{nb2, out, p->b ? out + nb2 : nullptr, p->c ? out + 2 * nb2 : nullptr};
  return RT_OK;
}

// pc (else NULL): block maxima of the componentwise measure
int finalize(rt_ctx* ctx, const Work& W, int op, int np, const double* pa, const double* pb,
             const double* pc = nullptr, int slot = 0) {
  const bool in_loop = op == FIN_ALPHA || op == FIN_BETA;
  Partials p{np, pa, pb, pc};
  RT_CHECK(fold(ctx, W, &p, W.partF,
                in_loop ? W.stop + (op == FIN_BETA ? STOP_P : STOP_X) : nullptr));
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kBlock), 0, ctx->stream, op, p.np, p.a, p.b, p.c,
                     W.scal, W.stop, slot);
  RT_LAUNCH_CHECK();
  return RT_OK;
}

// residual partials (npr of pr and pc), with pb also ||b||^2 (npb partials)
int start(rt_ctx* ctx, const Work& W, int npr, const double* pr, const double* pc, int npb,
          const double* pb, const int32_t* mismatch, const Tolerances& t) {
  Partials a{npr, pr, nullptr, pc}, b{npb, pb, nullptr, nullptr};
  RT_CHECK(fold(ctx, W, &a, W.partF, nullptr));
  if (pb) RT_CHECK(fold(ctx, W, &b, W.partF + 3 * kMaxPartials, nullptr));
  hipLaunchKernelGGL(k_start, dim3(1), dim3(kBlock), 0, ctx->stream, a.np, a.a, a.c, b.np, b.a,
                     mismatch, t, W.scal, W.stop);
  RT_LAUNCH_CHECK();
  return RT_OK;
}

// Componentwise test of a PCG loop: the update kernel's measure (mode) and its
// weights; the threshold is s[S_CWTHR] (infinity: measured, never binding).
struct CwTest {
  int mode = CW_NONE;
  const void* w = nullptr;
};

// p = z + beta p, beta from np partials (partA, partB, pc), or from the
// scalars when np = 0
template <typename T>
int pupdate(rt_ctx* ctx, rt_matrix* A, const Work& W, bool amg, int np, const double* pc, int slot,
            const T* r) {
  using S = Sel<T>;
  const Level& L = A->levels[0];
  const int gv = vec_blocks(L.n);
#define RT_PUPD(JAC_, E_)                                                                        \
  hipLaunchKernelGGL((k_pupdate<T, JAC_, E_>), dim3(gv), dim3(kBlock), 0, ctx->stream, L.n, np,   \
                     W.partA, W.partB, pc, slot, W.scal, r, JAC_ ? S::dinv(L) : nullptr,          \
                     JAC_ ? nullptr : S::z(W), S::p(W), W.stop)
  const bool one = vec_per_thread(L.n) == 1;
  if (amg && one) RT_PUPD(false, 1);
  else if (amg) RT_PUPD(false, kVec);
  else if (one) RT_PUPD(true, 1);
  else RT_PUPD(true, kVec);
#undef RT_PUPD
  RT_LAUNCH_CHECK();
  return RT_OK;
}

// One PCG iteration, queued; a no-op on the device once the stop flag is set.
// slot: the place of r.z it starts from (0, 1, 0, ... over the loop).
template <typename T>
int pcg_iteration(rt_ctx* ctx, rt_matrix* A, const Work& W, bool amg, T* x, T* r, const CwTest& cw,
                  int slot) {
  using S = Sel<T>;
  hipStream_t st = ctx->stream;
  const Level& L = A->levels[0];
  const int64_t n = L.n;
  T* p = S::p(W);
  T* q = S::q(W);
  T* z = S::z(W);
  int32_t* stop = W.stop;
  const int32_t* stop_p = W.stop + STOP_P;
  const int gv = vec_blocks(n);
  int nbk = 0;
  Prof pf(ctx, S::kind);
  RT_CHECK(pf.begin());
  const bool pair = pair_serves(L, level_shape<T>(L));
  if (pair)
    RT_CHECK((launch_pair<T, PP_DOT>(st, L, S::diag(L), p, q, W.partD, &nbk, level_shape<T>(L),
                                     nullptr, stop + STOP_X)));
  else
    RT_CHECK((launch_spmv_level<T, SP_DOT>(st, L, S::val(L), S::diag(L), p, nullptr, nullptr, q,
                                           nullptr, W.partD, &nbk, level_shape<T>(L), nullptr,
                                           stop + STOP_X)));
  RT_CHECK(pf.end());
  // the product's partials go to partD, so that the update's blocks can read
  // them while others already write theirs
  const bool fa = nbk <= RT_FUSED_PARTIALS, fb = gv <= kFusedVec;
  if (!fa) RT_CHECK(finalize(ctx, W, FIN_ALPHA, nbk, W.partD, nullptr, nullptr, slot));
  const T* w = static_cast<const T*>(cw.w);
  double* pc = cw.mode == CW_NONE ? nullptr : W.partC;
#define RT_UPD1(JAC_, CW_, PAIR_, E_)                                                           \
  hipLaunchKernelGGL((k_update<T, JAC_, CW_, PAIR_, E_>), dim3(gv), dim3(kBlock), 0, st, n,      \
                     L.pair.in(), PairSel<T>::sum(L.pair), fa ? nbk : 0, W.partD, slot, W.scal, x, \
                     r, p, q,                                                                    \
                     JAC_ ? S::dinv(L) : nullptr, w, W.partA, JAC_ ? W.partB : nullptr, pc, stop)
  const bool one = vec_per_thread(n) == 1;
#define RT_UPD(JAC_, CW_)                            \
  do {                                               \
    if (pair && one) RT_UPD1(JAC_, CW_, true, 1);    \
    else if (pair) RT_UPD1(JAC_, CW_, true, kVec);   \
    else if (one) RT_UPD1(JAC_, CW_, false, 1);      \
    else RT_UPD1(JAC_, CW_, false, kVec);            \
  } while (0)
  if (amg) {
    if (cw.mode == CW_X) RT_UPD(false, CW_X);
    else if (cw.mode == CW_W) RT_UPD(false, CW_W);
    else RT_UPD(false, CW_NONE);
    RT_LAUNCH_CHECK();
    RT_CHECK(vcycle<T>(ctx, A, r, z, stop_p));
    hipLaunchKernelGGL(k_dot<T>, dim3(gv), dim3(kBlock), 0, st, n, r, z, W.partB, stop_p);
  } else {
    if (cw.mode == CW_X) RT_UPD(true, CW_X);
    else if (cw.mode == CW_W) RT_UPD(true, CW_W);
    else RT_UPD(true, CW_NONE);
  }
#undef RT_UPD
#undef RT_UPD1
  RT_LAUNCH_CHECK();
  if (!fb) RT_CHECK(finalize(ctx, W, FIN_BETA, gv, W.partA, W.partB, pc, slot));
  RT_CHECK(pupdate<T>(ctx, A, W, amg, fb ? gv : 0, pc, slot, r));
  return RT_OK;
}

// Iterations to queue before the next read of the state, from the decrease
// of ||r||^2 since the last read: three quarters of the estimated remaining
// count (at least one, at most 64); one while there is no decrease to go by.
int next_chunk(double rr_prev, int its_prev, double rr, int its, double thr2) {
  if (!(its > its_prev) || !(rr > 0.0) || !(rr < rr_prev) || !(thr2 > 0.0)) return 1;
  const double per_it = std::log(rr / rr_prev) / (its - its_prev);   // < 0
  const double need = std::log(thr2 / rr) / per_it;                  // > 0
  if (!std::isfinite(need)) return 1;
  return (int)std::min(64.0, std::max(1.0, std::floor(0.75 * need)));
}

// What a loop found and did, read back from the device scalars.
struct LoopState {
  double bb = 0.0, rr0 = 0.0, cw0 = 0.0;   // at its start (k_start)
  double rr = 0.0, cw = 0.0;               // at its end
  int its = 0;
  bool done = false, mismatch = false, bad = false;
};
int read_state(rt_ctx* ctx, const Work& W, LoopState* s) {
  RT_CHECK(ctx->sync_read(W.scal, sizeof(double) * S_COUNT));
  const double* h = ctx->host;
  s->bb = h[S_BB];
  s->rr0 = h[S_RR0];
  s->cw0 = h[S_CW0];
  s->rr = h[S_RR];
  s->cw = h[S_CW];
  s->its = (int)h[S_ITS];
  s->done = h[S_DONE] != 0.0;
  s->mismatch = h[S_MIS] != 0.0;
  s->bad = h[S_BAD] != 0.0;
  return RT_OK;
}

// PCG iterations on A x = b given r = b - A x, after start() has set the
// thresholds: until the device stops or max_it iterations ran.  first: the
// iterations queued before the first read of the state.
template <typename T>
int pcg_core(rt_ctx* ctx, rt_matrix* A, const Work& W, bool amg, T* x, T* r, int max_it,
             const CwTest& cw, int first, bool resume, LoopState* out) {
  using S = Sel<T>;
  hipStream_t st = ctx->stream;
  const Level& L = A->levels[0];
  const int64_t n = L.n;
  T* p = S::p(W);
  T* z = S::z(W);
  const int gv = vec_blocks(n);
  *out = LoopState{};
  if (max_it <= 0) return read_state(ctx, W, out);
  if (amg) {
    // A loop that ends where it starts (the last outer iteration of a step, the
    // last refinement) would run dozens of launches of a V-cycle for nothing.
    RT_CHECK(read_state(ctx, W, out));
    if (ctx->host[S_STOP] != 0.0) return RT_OK;
    RT_CHECK(vcycle<T>(ctx, A, r, z, W.stop));
  }
  if (resume) {
    // the last loop on this system ended at a residual replacement: its
    // search direction p carries over, p = z + beta p with the new r.z
    if (amg)
      hipLaunchKernelGGL(k_dot<T>, dim3(gv), dim3(kBlock), 0, st, n, r, z, W.partB, W.stop);
    else
      hipLaunchKernelGGL(k_rz_jacobi<T>, dim3(gv), dim3(kBlock), 0, st, n, S::dinv(L), r, W.partB,
                         W.stop);
    RT_LAUNCH_CHECK();
    RT_CHECK(finalize(ctx, W, FIN_RESUME, gv, W.partB, nullptr));
    RT_CHECK(pupdate<T>(ctx, A, W, amg, 0, nullptr, 0, r));
  } else {
    if (amg)
      hipLaunchKernelGGL(k_copy_dot<T>, dim3(gv), dim3(kBlock), 0, st, n, r, z, p, W.partB, W.stop);
    else
      hipLaunchKernelGGL(k_init_jacobi<T>, dim3(gv), dim3(kBlock), 0, st, n, S::dinv(L), r, p,
                         W.partB, W.stop);
    RT_LAUNCH_CHECK();
    RT_CHECK(finalize(ctx, W, FIN_RZ, gv, W.partB, nullptr));
  }
  const size_t spans0 = ctx->prof_spans.size();
  double rr_prev = 0.0;
  int its_prev = 0, queued = 0, chunk = first;
  while (queued < max_it) {
    const int k = std::min(chunk, max_it - queued);
    for (int j = 0; j < k; ++j)
      RT_CHECK(pcg_iteration<T>(ctx, A, W, amg, x, r, cw, (queued + j) & 1));
    const bool start_read = queued == 0;
    queued += k;
    RT_CHECK(read_state(ctx, W, out));
    if (start_read) rr_prev = out->rr0;
    if (out->its > 0 && !std::isfinite(out->rr)) {
      set_error("PCG breakdown: non-finite residual");
      return RT_E_DEVICE;
    }
    if (ctx->host[S_STOP] != 0.0) break;
    // while the componentwise test still binds, go by one iteration at a time
    const double thr2 = ctx->host[S_THR];
    chunk = out->rr > thr2 ? next_chunk(rr_prev, its_prev, out->rr, out->its, thr2) : 1;
    // an estimate from few iterations is often far too long: at most double
    chunk = std::min(chunk, std::max(2, out->its));
    rr_prev = out->rr;
    its_prev = out->its;
  }
  if (out->bad && out->rr > ctx->host[S_THR])
    set_error("PCG breakdown: p.Ap not positive after %d iterations", out->its);
  // product timings of queued iterations that did not run are dropped
  if (ctx->profiling && ctx->prof_spans.size() > spans0 + (size_t)out->its)
    ctx->prof_spans.resize(spans0 + (size_t)out->its);
  return RT_OK;
}

int ensure_work(rt_matrix* A, bool mixed) {
  const int64_t n = A->n;
  for (auto* b : {&A->r64, &A->p64, &A->q64, &A->z64}) RT_CHECK(b->reserve(n));
  RT_CHECK(A->partA.reserve(max_partials(n)));
  RT_CHECK(A->partB.reserve(max_partials(n)));
  RT_CHECK(A->partC.reserve(max_partials(n)));
  RT_CHECK(A->partD.reserve(max_partials(n)));
  RT_CHECK(A->partF.reserve(6 * kMaxPartials));
  RT_CHECK(A->scal.reserve(std::max<int>(S_COUNT, kScalars)));
  RT_CHECK(A->stop.reserve(STOP_WORDS));
  if (mixed)
    for (auto* b : {&A->r32, &A->p32, &A->q32, &A->z32, &A->d32, &A->w32}) RT_CHECK(b->reserve(n));
  return RT_OK;
}

// The CSR rows of a level in pair form, when a plain shape asks for them.
int ensure_shapes(rt_ctx* ctx, rt_matrix* A, bool mixed) {
  const Level& L = A->levels[0];
  return wants_rows(L, mixed ? L.shape32 : L.shape64) ? ensure_csr(ctx, A) : RT_OK;
}

// The matrix's own work buffers (after ensure_work)
Work work_of(rt_matrix* A) {
  Work W;
  W.r64 = A->r64.p;
  W.p64 = A->p64.p;
  W.q64 = A->q64.p;
  W.z64 = A->z64.p;
  W.r32 = A->r32.p;
  W.p32 = A->p32.p;
  W.q32 = A->q32.p;
  W.z32 = A->z32.p;
  W.d32 = A->d32.p;
  W.w32 = A->w32.p;
  W.partA = A->partA.p;
  W.partB = A->partB.p;
  W.partC = A->partC.p;
  W.partD = A->partD.p;
  W.partF = A->partF.p;
  W.scal = A->scal.p;
  W.stop = A->stop.p;
  return W;
}

// r = b - A x in FP64 (optionally also r32 and the componentwise weights
// w32), with *nparts partials of ||r||^2 and of the componentwise measure
// max_i |r_i| / (a_ii |x_i|) in partA and partC
int residual64(rt_ctx* ctx, rt_matrix* A, const Work& W, const double* b, const double* x, float* r32,
               float* w32, int* nparts) {
  const Level& L = A->levels[0];
  Prof pf(ctx, PROF_RESID64);
  RT_CHECK(pf.begin());
  if (pair_serves(L, resid_shape(L)))
    RT_CHECK(pair_resid(ctx, L, x, b, W.r64, r32, w32, W.partA, W.partC, nparts, resid_shape(L)));
  else
    RT_CHECK((launch_spmv_level<double, SP_RESID>(ctx->stream, L, L.val64.p, L.diag64.p, x, b,
                                                  nullptr, W.r64, r32, W.partA, nparts,
                                                  resid_shape(L), nullptr, nullptr, W.partC, w32)));
  return pf.end();
}

// FP64 CG steps after which the recursive residual is replaced by a
// computed one: the recursion's drift from b - A x grows with the steps
// taken (and carried between outer iterations); one product per 32 steps
// keeps it at rounding level for about 3% more products on long solves.
constexpr int kReplaceSteps = 32;

// The solve on sorted vectors with the buffers of W (see solve_sorted);
// *resid_valid: W.r64 holds b - A x on return.  *rec_steps: on entry, the
// CG steps the residual carried in W.r64 (with b_prev) has been updated by
// recursion since a product formed it; on return, the same for W.r64.
int solve_work(rt_ctx* ctx, rt_matrix* A, const Work& W, const double* b, double* x,
               const rt_solve_opts* o, rt_solve_stats* stt, const double* b_prev,
               const int32_t* mismatch, bool* resid_valid, int* rec_steps) {
  hipStream_t st = ctx->stream;
  const int64_t n = A->n;
  const bool mixed = o->precision == RT_PREC_MIXED;
  *resid_valid = false;
  const bool amg = o->precond == 1 && cycle_depth(A) > 1;
  *stt = rt_solve_stats{};
  if (n == 0) return RT_OK;
  const int gv = vec_blocks(n);
  const Level& L0 = A->levels[0];
  // componentwise test: its threshold, infinity when only measured
  const bool use_cw = o->cw_tol > 0.0;
  const double cwthr = use_cw ? o->cw_tol : INFINITY;
  float* r32 = mixed ? W.r32 : nullptr;
  float* w32 = mixed && use_cw ? W.w32 : nullptr;
  const Tolerances t{o->tol * o->tol, cwthr, mixed ? o->inner_tol : 0.0};
  const CwTest cwt = mixed ? (use_cw ? CwTest{CW_W, w32} : CwTest{}) : CwTest{CW_X, L0.dinv64.p};
  if (mixed) {
    hipLaunchKernelGGL(k_zero<float>, dim3(grid_for(n)), dim3(kBlock), 0, st, n, W.d32);
    RT_LAUNCH_CHECK();
  }
  // one inner loop (a whole solve in FP64) on the residual that start() saw
  auto loop = [&](int max_it, int first, bool resume, LoopState* ls) {
    return mixed ? pcg_core<float>(ctx, A, W, amg, W.d32, W.r32, max_it, cwt, first, resume, ls)
                 : pcg_core<double>(ctx, A, W, amg, x, W.r64, max_it, cwt, first, resume, ls);
  };
  // the first residual: the last one shifted by the change of b, or a product
  bool shifted = b_prev != nullptr;
  int nbk = 0;
  LoopState ls;
  const int first = mixed ? 2 : 3;
  for (;;) {
    if (shifted) {
      hipLaunchKernelGGL(k_resid_shift, dim3(gv), dim3(kBlock), 0, st, n, b, b_prev, x,
                         L0.diag64.p, W.r64, r32, w32, W.partA, W.partB, W.partC);
      RT_LAUNCH_CHECK();
      RT_CHECK(start(ctx, W, gv, W.partA, W.partC, gv, W.partB, mismatch, t));
    } else {
      hipLaunchKernelGGL(k_dot<double>, dim3(gv), dim3(kBlock), 0, st, n, b, b, W.partB, nullptr);
      RT_LAUNCH_CHECK();
      RT_CHECK(residual64(ctx, A, W, b, x, r32, w32, &nbk));
      RT_CHECK(start(ctx, W, nbk, W.partA, W.partC, gv, W.partB, nullptr, t));
    }
    const int s = loop(mixed && o->max_refine <= 0 ? 0 : o->max_iter, first, false, &ls);
    if (std::isfinite(ls.bb) && s < 0) return s;
    if (!ls.mismatch) break;
    shifted = false;   // E^l is not the last solution: form the residual
  }
  const double bb = ls.bb;
  if (!std::isfinite(bb)) {
    set_error("rt_solve: right-hand side is not finite");
    return RT_E_ARG;
  }
  if (bb == 0.0) {
    hipLaunchKernelGGL(k_zero<double>, dim3(grid_for(n)), dim3(kBlock), 0, st, n, x);
    RT_LAUNCH_CHECK();
    return RT_OK;
  }
  const double thr2 = o->tol * o->tol * bb;
  stt->init_rel_residual = std::sqrt(ls.rr0 / bb);
  int status = RT_OK;
  double rr = ls.rr, cw = ls.cw;
  if (!mixed) {
    int rec = shifted ? *rec_steps : 0;
    int total = ls.its;
    rec += ls.its;
    for (int pass = 0; rec > kReplaceSteps && pass < 2; ++pass) {
      // residual replacement; CG restarts from the computed residual if it
      // misses the tolerance
      RT_CHECK(residual64(ctx, A, W, b, x, nullptr, nullptr, &nbk));
      RT_CHECK(start(ctx, W, nbk, W.partA, W.partC, 0, nullptr, nullptr, t));
      rec = 0;
      ++stt->replacements;
      RT_CHECK(loop(o->max_iter - total, first, false, &ls));
      rr = ls.rr;
      cw = ls.cw;
      total += ls.its;
      rec += ls.its;
      if (ls.done || total >= o->max_iter) break;
    }
    stt->iterations = total;
    *rec_steps = rec;
  } else {
    *rec_steps = 0;
    int total = 0, refine = 0;
    // After the first inner solve each one continues the last: the FP64
    // residual replaces CG's recursive one (reliable update) and the search
    // direction carries over, so the refinements do not restart the Krylov
    // space.
    rr = ls.rr0;
    cw = ls.cw0;
    while (!ls.done && total < o->max_iter && refine < o->max_refine) {
      const int its = ls.its;
      total += its;
      hipLaunchKernelGGL(k_add_f32, dim3(grid_for(n)), dim3(kBlock), 0, st, n, W.d32, x);
      RT_LAUNCH_CHECK();
      RT_CHECK(residual64(ctx, A, W, b, x, W.r32, w32, &nbk));
      RT_CHECK(start(ctx, W, nbk, W.partA, W.partC, 0, nullptr, nullptr, t));
      ++refine;
      // the next inner loop, queued before the host knows whether it is needed
      const bool more = its > 0 && total < o->max_iter && refine < o->max_refine;
      RT_CHECK(loop(more ? o->max_iter - total : 0, first, its > 0, &ls));
      rr = ls.rr0;
      cw = ls.cw0;
      if (!more) break;
    }
    stt->iterations = total;
    stt->refinements = refine;
  }
  if (rr > thr2 || cw > cwthr) status = RT_NOT_CONVERGED;
  stt->rel_residual = std::sqrt(rr / bb);
  stt->cw_residual = cw;
  // r64 now holds b - A x: the residual of an FP64 product (mixed), or the
  // recursive residual of CG (FP64), which differs from it by rounding only
  *resid_valid = true;
  if (status == RT_NOT_CONVERGED)
    set_error("rt_solve: relative residual %.3e (componentwise %.3e) above tolerance %.3e "
              "(componentwise %.3e)", stt->rel_residual, cw, o->tol, o->cw_tol);
  return status;
}

}  // namespace

int residual_norms(rt_ctx* ctx, rt_matrix* A, const double* b, const double* x, double* rr,
                   double* bb) {
  A->resid_ok = false;
  A->r64_valid = false;
  RT_CHECK(ensure_work(A, false));
  RT_CHECK(ensure_shapes(ctx, A, true));
  const Work W = work_of(A);
  int nbk = 0;
  RT_CHECK(residual64(ctx, A, W, b, x, nullptr, nullptr, &nbk));
  RT_CHECK(finalize(ctx, W, FIN_RR, nbk, W.partA, nullptr, W.partC));
  const int gv = vec_blocks(A->n);
  hipLaunchKernelGGL(k_dot<double>, dim3(gv), dim3(kBlock), 0, ctx->stream, A->n, b, b, W.partB,
                     nullptr);
  RT_LAUNCH_CHECK();
  RT_CHECK(finalize(ctx, W, FIN_BB, gv, W.partB, nullptr));
  LoopState ls;
  RT_CHECK(read_state(ctx, W, &ls));
  *rr = ls.rr;
  *bb = ls.bb;
  return RT_OK;
}

int solve_sorted(rt_ctx* ctx, rt_matrix* A, const double* b, double* x, const rt_solve_opts* o,
                 rt_solve_stats* stt, const double* b_prev, const int32_t* mismatch) {
  const bool mixed = o->precision == RT_PREC_MIXED;
  A->r64_valid = false;
  if (mixed && !A->has_fp32) {
    set_error("rt_solve: mixed precision needs a matrix assembled with build_fp32 = 1");
    return RT_E_STATE;
  }
  RT_CHECK(ensure_work(A, mixed));
  RT_CHECK(ensure_shapes(ctx, A, mixed));
  bool valid = false;
  int rec = A->rec_steps;
  const int s = solve_work(ctx, A, work_of(A), b, x, o, stt, b_prev, mismatch, &valid, &rec);
  A->r64_valid = valid;
  A->rec_steps = rec;
  return s;
}

int collect_profile(rt_ctx* ctx, rt_solve_stats* s) {
  if (!ctx->profiling) return RT_OK;
  double sec[PROF_KINDS];
  int calls[PROF_KINDS];
  RT_CHECK(ctx->prof_collect(sec, calls, PROF_KINDS));
  s->spmv_calls = calls[PROF_SPMV64];
  s->spmv_seconds = sec[PROF_SPMV64];
  s->spmv32_calls = calls[PROF_SPMV32];
  s->spmv32_seconds = sec[PROF_SPMV32];
  s->resid_calls = calls[PROF_RESID64];
  s->resid_seconds = sec[PROF_RESID64];
  return RT_OK;
}

int gather_sorted(rt_ctx* ctx, const rt_neighbors* nb, int64_t n, const double* user,
                  double* sorted) {
  hipLaunchKernelGGL(k_gather, dim3(grid_for(n)), dim3(kBlock), 0, ctx->stream, n, nb->perm.p,
                     user, sorted);
  RT_LAUNCH_CHECK();
  return RT_OK;
}

int scatter_user(rt_ctx* ctx, const rt_neighbors* nb, int64_t n, const double* sorted,
                 double* user) {
  hipLaunchKernelGGL(k_scatter, dim3(grid_for(n)), dim3(kBlock), 0, ctx->stream, n, nb->perm.p,
                     sorted, user);
  RT_LAUNCH_CHECK();
  return RT_OK;
}

int check_solve_opts(const rt_solve_opts* o) {
  if (!o) {
    set_error("solve options are NULL");
    return RT_E_ARG;
  }
  if (o->precision != RT_PREC_FP64 && o->precision != RT_PREC_MIXED) {
    set_error("unknown precision %d", o->precision);
    return RT_E_ARG;
  }
  if (o->precond != 0 && o->precond != 1) {
    set_error("unknown preconditioner %d", o->precond);
    return RT_E_ARG;
  }
  if (!(o->tol >= 0.0) || o->max_iter < 0 || !(o->cw_tol >= 0.0) ||
      (o->precision == RT_PREC_MIXED && (!(o->inner_tol > 0.0) || o->inner_tol >= 1.0))) {
    set_error("invalid tolerance or iteration limit");
    return RT_E_ARG;
  }
  return RT_OK;
}

}  // namespace rt

namespace rt {
namespace {

// Largest systems of the no-allocation solve.
constexpr int64_t kScratchMaxFp64 = 4968256, kScratchMaxMixed = 3439552;

// Bytes of scratch the no-allocation solve carves for n unknowns: the gathered
// b and x, four FP64 work vectors (six FP32 ones in mixed precision), four
// arrays of block partials, the fold buffer, the scalars and the stop flag,
// each piece 256-byte aligned.
struct Carve {
  char* base;
  size_t used = 0;
  template <typename T>
  T* take(size_t count) {
    used = (used + 255) / 256 * 256;
    T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
    used += (count ? count : 1) * sizeof(T);
    return p;
  }
};

Work carve_work(Carve& c, int64_t n, bool mixed, double** bs, double** xs) {
  Work W;
  *bs = c.take<double>(n);
  *xs = c.take<double>(n);
  W.r64 = c.take<double>(n);
  W.p64 = c.take<double>(n);
  W.q64 = c.take<double>(n);
  W.z64 = c.take<double>(n);
  if (mixed) {
    W.r32 = c.take<float>(n);
    W.p32 = c.take<float>(n);
    W.q32 = c.take<float>(n);
    W.z32 = c.take<float>(n);
    W.d32 = c.take<float>(n);
    W.w32 = c.take<float>(n);
  }
  // partials of products (at most one per four rows) and of vector passes
  for (double** p : {&W.partA, &W.partC, &W.partD}) *p = c.take<double>(spmv_blocks(n, 64));
  W.partB = c.take<double>(vec_blocks(n));
  W.partF = c.take<double>(6 * kMaxPartials);
  W.scal = c.take<double>(S_COUNT);
  W.stop = c.take<int32_t>(STOP_WORDS);
  return W;
}

}  // namespace
}  // namespace rt

// rt_solve for callers that cannot allocate: every buffer of the solve comes
// from the device's scratch array; the matrix's own work buffers and the
// residual it carries between outer iterations are left untouched.
extern "C" int rt_solve_noalloc(rt_ctx* ctx, rt_matrix* A, const double* b, double* x,
                                const rt_solve_opts* opts, rt_solve_stats* stats) {
  using namespace rt;
  clear_error();
  if (!ctx || !A || (A->n > 0 && (!b || !x))) {
    set_error("rt_solve_noalloc: NULL argument");
    return RT_E_ARG;
  }
  RT_CHECK(check_solve_opts(opts));
  if (A->levels.empty()) {
    set_error("rt_solve_noalloc: matrix not assembled");
    return RT_E_STATE;
  }
  const bool mixed = opts->precision == RT_PREC_MIXED;
  if (mixed && !A->has_fp32) {
    set_error("rt_solve_noalloc: mixed precision needs a matrix assembled with build_fp32 = 1");
    return RT_E_STATE;
  }
  const int64_t n = A->n;
  Carve size{nullptr};
  double *bs = nullptr, *xs = nullptr;
  (void)carve_work(size, n, mixed, &bs, &xs);
  // the documented limits (the pieces just fit the array at them)
  const int64_t most = mixed ? kScratchMaxMixed : kScratchMaxFp64;
  if (n > most || size.used > kScratchBytes) {
    set_error("rt_solve_noalloc: %lld unknowns need %zu bytes of scratch in %s, above the "
              "%zu-byte scratch array", (long long)n, size.used,
              mixed ? "mixed precision" : "FP64", kScratchBytes);
    return RT_E_ARG;
  }
  RT_CHECK_HIP(hipSetDevice(ctx->device));
  char* base = static_cast<char*>(scratch_base(ctx->device));
  if (!base) {
    set_error("rt_solve_noalloc: no scratch address for device %d", ctx->device);
    return RT_E_STATE;
  }
  auto t0 = std::chrono::steady_clock::now();
  rt_solve_stats local{};
  rt_solve_stats* stt = stats ? stats : &local;
  *stt = rt_solve_stats{};
  if (n == 0) return RT_OK;
  Carve carve{base};
  const Work W = carve_work(carve, n, mixed, &bs, &xs);
  // no event timings: recording them would create events
  const bool prof = ctx->profiling;
  ctx->profiling = false;
  int s = gather_sorted(ctx, A->nb, n, b, bs);
  if (s == RT_OK) s = gather_sorted(ctx, A->nb, n, x, xs);
  bool valid = false;
  int rec = 0;
  if (s == RT_OK) s = solve_work(ctx, A, W, bs, xs, opts, stt, nullptr, nullptr, &valid, &rec);
  ctx->profiling = prof;
  if (s < 0) return s;
  RT_CHECK(scatter_user(ctx, A->nb, n, xs, x));
  RT_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  stt->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return s;
}

extern "C" int rt_solve(rt_ctx* ctx, rt_matrix* A, const double* b, double* x,
                        const rt_solve_opts* opts, rt_solve_stats* stats) {
  using namespace rt;
  clear_error();
  if (!ctx || !A || (A->n > 0 && (!b || !x))) {
    set_error("rt_solve: NULL argument");
    return RT_E_ARG;
  }
  RT_CHECK(check_solve_opts(opts));
  RT_CHECK_HIP(hipSetDevice(ctx->device));
  rt::StreamScope release_scope(ctx->stream);   // buffers released here are stream-ordered
  auto t0 = std::chrono::steady_clock::now();
  rt_solve_stats local{};
  rt_solve_stats* stt = stats ? stats : &local;
  A->resid_ok = false;   // bs, xs and r64 are overwritten here
  RT_CHECK(A->xs.reserve(A->n));
  RT_CHECK(A->bs.reserve(A->n));
  RT_CHECK(gather_sorted(ctx, A->nb, A->n, b, A->bs.p));
  RT_CHECK(gather_sorted(ctx, A->nb, A->n, x, A->xs.p));
  int s = solve_sorted(ctx, A, A->bs.p, A->xs.p, opts, stt);
  if (s < 0) return s;
  RT_CHECK(scatter_user(ctx, A->nb, A->n, A->xs.p, x));
  RT_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  RT_CHECK(collect_profile(ctx, stt));
  stt->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return s;
}
