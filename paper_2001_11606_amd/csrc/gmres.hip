// Restarted GMRES on the unscaled diffusion operator, as the paper solves the
// diffusion equation (Sec. 3.2, with a multigrid preconditioner).
//
// The library's main solver is CG on the V-scaled symmetric system A x = b
// (row i of the paper's operator multiplied by V_i).  This solver works on
// the paper's own, unscaled form U x = c with U = diag(V)^-1 A and
// c = diag(V)^-1 b, which has the same solution x.  U is not symmetric.
//
// Right-preconditioned GMRES(m): the Krylov space is built from U M^-1 and
// x = x0 + M^-1 (Z y), so the residual the method minimises is the true
// residual of U x = c.  The preconditioner approximates U^-1 = A^-1 diag(V):
//   Jacobi:  M^-1 v = diag(A)^-1 (V v)   (= diag(U)^-1 v)
//   AMG:     M^-1 v = Vcycle(V v)        (the V-cycle of A)
// Both are linear and fixed, so the correction is formed once per cycle from
// the combined basis vector.  The basis is orthogonalised by classical
// Gram-Schmidt applied twice; the small Hessenberg least-squares problem is
// solved on the host with Givens rotations.  Stop when ||c - U x||_2 <= tol
// ||c||_2; the final relative residual is recomputed from a product, not taken
// from the recurrence.  FP64 throughout.
//
// An iteration is a product and three passes over the basis, each of which
// also forms what the next step needs (k_g_dots: w = (A z)/V and its dots;
// k_g_project: w minus its projection and the dots of the second pass;
// k_g_last: the second projection and the norm), with small reductions
// between them.  The coefficients stay on the device, and the host reads the
// columns of several iterations at a time; columns past the one that
// converges are dropped.  The basis passes are bound by the reads of the basis
// (2.9 TB/s and up, from the last-level cache at 262k rows, 18 vectors on
// average); a solve of 36 iterations there takes 2.6 ms, and 6.1 ms with a
// host read per dot product and eleven launches an iteration.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "internal.h"
#include "reduce.h"
#include "pair.h"
#include "spmv.h"

namespace rt {
namespace {

constexpr int kGmresMaxRestart = 64;
constexpr int kGmresCol = kGmresMaxRestart + 2;   // stride of the Hessenberg columns on the device

// Elements per thread of the basis passes: one up to this size, so that the
// grid fills the chip, four beyond, where the partials of one per thread cost
// more.  A density-step solve with one | four: 262k rows 2.6 | 3.4 ms, 512k
// 4.9 | 5.3, 1.03M 9.7 | 8.8, 2.1M 25.3 | 23.4.
constexpr int64_t kGmresOne = (int64_t)3 << 18;
#define RT_G_LOOP(i, e)                                                                       \
  for (int e = 0; e < E; ++e)                                                                 \
    for (int64_t i = ((int64_t)blockIdx.x * E + e) * kBlock + threadIdx.x; i < n; i = n)

// Block partials are kept per wave: part[j * nw + wave], no barrier between
// the dots of consecutive basis vectors.
template <int E>
__device__ __forceinline__ void g_dots(int64_t n, int J, const double* __restrict__ basis,
                                       const double* w, int64_t nw, double* __restrict__ part) {
  const int64_t wave = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  int j = 0;
  for (; j + 3 < J; j += 4) {   // four vectors in flight
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    RT_G_LOOP(i, e) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += w[e] * basis[(int64_t)(j + u) * n + i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc[u] = group_sum<kWave>(acc[u]);
      if ((threadIdx.x & (kWave - 1)) == 0) part[(int64_t)(j + u) * nw + wave] = acc[u];
    }
  }
  for (; j < J; ++j) {
    double acc = 0.0;
    RT_G_LOOP(i, e) acc += w[e] * basis[(int64_t)j * n + i];
    acc = group_sum<kWave>(acc);
    if ((threadIdx.x & (kWave - 1)) == 0) part[(int64_t)j * nw + wave] = acc;
  }
}

// w = (t + the sums earlier tiles left) / V, and the partials of w . basis_j, j < J
template <int E, bool PAIR>
__global__ void __launch_bounds__(kBlock)
k_g_dots(int64_t n, int J, PairIn P, const double* __restrict__ tsum, const double* __restrict__ t,
         const double* __restrict__ V, const double* __restrict__ basis, double* __restrict__ w,
         int64_t nw, double* __restrict__ part) {
  double we[E];
#pragma unroll
  for (int e = 0; e < E; ++e) we[e] = 0.0;
  RT_G_LOOP(i, e) {
    double ti = t[i];
    if (PAIR) ti += pair_in<double>(P, i, tsum);
    we[e] = ti / V[i];
    w[i] = we[e];
  }
  g_dots<E>(n, J, basis, we, nw, part);
}

// w -= sum_j c_j basis_j; then the partials of w . basis_j (DOTS) or of w . w
template <int E, bool DOTS>
__global__ void __launch_bounds__(kBlock)
k_g_project(int64_t n, int J, const double* __restrict__ c, const double* __restrict__ basis,
            double* __restrict__ w, int64_t nw, double* __restrict__ part) {
  double we[E];
#pragma unroll
  for (int e = 0; e < E; ++e) we[e] = 0.0;
#pragma unroll 8
  for (int j = 0; j < J; ++j) {
    const double cj = c[j];
    RT_G_LOOP(i, e) we[e] += cj * basis[(int64_t)j * n + i];
  }
  RT_G_LOOP(i, e) {
    we[e] = w[i] - we[e];
    w[i] = we[e];
  }
  if (DOTS) {
    g_dots<E>(n, J, basis, we, nw, part);
  } else {
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) acc += we[e] * we[e];
    acc = group_sum<kWave>(acc);
    if ((threadIdx.x & (kWave - 1)) == 0)
      part[((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave] = acc;
  }
}

// w = in / V and the partials of w . w
template <int E>
__global__ void __launch_bounds__(kBlock)
k_g_div_norm(int64_t n, const double* __restrict__ in, const double* __restrict__ V,
             double* __restrict__ w, double* __restrict__ part) {
  double acc = 0.0;
  RT_G_LOOP(i, e) {
    const double x = in[i] / V[i];
    w[i] = x;
    acc += x * x;
  }
  acc = group_sum<kWave>(acc);
  if ((threadIdx.x & (kWave - 1)) == 0)
    part[((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave] = acc;
}

// Block j: c[j] = the sum of row j of the partials; h[j] = c[j] (first) or
// h[j] += c[j]; root: c[0] = h[0] = its square root (a norm).
__global__ void __launch_bounds__(kBlock)
k_g_reduce(int64_t nw, const double* __restrict__ part, int first, int root,
           double* __restrict__ c, double* __restrict__ h) {
  __shared__ double red[kBlock / kWave];
  const int j = blockIdx.x;
  const double* __restrict__ pj = part + (int64_t)j * nw;
  double a4[4] = {0.0, 0.0, 0.0, 0.0};
  int64_t i = threadIdx.x;
  for (; i + 3 * kBlock < nw; i += 4 * kBlock)
#pragma unroll
    for (int u = 0; u < 4; ++u) a4[u] += pj[i + u * kBlock];
  for (int u = 0; i < nw; i += kBlock, ++u) a4[u] += pj[i];
  double s = block_sum((a4[0] + a4[1]) + (a4[2] + a4[3]), red);
  if (threadIdx.x != 0) return;
  if (root) s = sqrt(s);
  c[j] = s;
  h[j] = first ? s : h[j] + s;
}

// v = w / *norm and what the preconditioner takes of it: z = s V v (Jacobi, s =
// 1/diag(A)) or z = V v (s NULL)
__global__ void __launch_bounds__(kBlock)
k_g_next(int64_t n, const double* __restrict__ norm, const double* w, const double* __restrict__ s,
         const double* __restrict__ V, double* v, double* __restrict__ z) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= n) return;
  const double x = w[i] * (1.0 / *norm);
  v[i] = x;
  z[i] = (s ? s[i] : 1.0) * (V[i] * x);
}

struct GCoef {
  double c[kGmresMaxRestart];
};

// u = sum_{j<J} c_j basis_j; x += s V u (Jacobi), or z = V u (s NULL)
__global__ void __launch_bounds__(kBlock)
k_g_combine(int64_t n, int J, GCoef C, const double* __restrict__ basis,
            const double* __restrict__ s, const double* __restrict__ V, double* __restrict__ x,
            double* __restrict__ z) {
  const int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x;
  if (i >= n) return;
  double u = 0.0;
  for (int j = 0; j < J; ++j) u += C.c[j] * basis[(int64_t)j * n + i];
  if (s) x[i] += s[i] * (V[i] * u);
  else z[i] = V[i] * u;
}

// x += z
__global__ void k_add(int64_t n, const double* __restrict__ z, double* __restrict__ x) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[i] += z[i];
}

__global__ void k_fill0(int64_t n, double* __restrict__ out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = 0.0;
}

struct Gmres {
  rt_ctx* ctx;
  rt_matrix* A;
  int64_t n;
  int m;
  bool amg;
  DevBuf<double> basis, w, t, z, part, coef, hess;
  int64_t nw = 1;   // waves (= partials per dot) of a basis pass
  int blocks = 1;
  bool one = true;

  int init() {
    one = n <= kGmresOne;
    blocks = grid_for(n, kBlock * (one ? 1 : 4));
    nw = (int64_t)blocks * (kBlock / kWave);
    RT_CHECK(basis.reserve((size_t)(m + 1) * n));
    for (auto* b : {&w, &t, &z}) RT_CHECK(b->reserve(n));
    RT_CHECK(part.reserve((size_t)(m + 1) * nw));
    RT_CHECK(coef.reserve(m + 2));
    RT_CHECK(hess.reserve((size_t)kGmresCol * (m + 1)));
    return RT_OK;
  }
  double* vec(int j) { return basis.p + (int64_t)j * n; }
  double* column(int k) { return hess.p + (int64_t)k * kGmresCol; }
  const double* jacobi() const { return amg ? nullptr : A->levels[0].dinv64.p; }
  int reduce(int J, bool first, bool root, double* h) {
    hipLaunchKernelGGL(k_g_reduce, dim3(J), dim3(kBlock), 0, ctx->stream, nw, part.p,
                       first ? 1 : 0, root ? 1 : 0, coef.p, h);
    RT_LAUNCH_CHECK();
    return RT_OK;
  }
  // w = in / V; *norm = ||w||, read back
  int div_norm(const double* in, double* norm) {
    if (one)
      hipLaunchKernelGGL(k_g_div_norm<1>, dim3(blocks), dim3(kBlock), 0, ctx->stream, n, in,
                         A->V.p, w.p, part.p);
    else
      hipLaunchKernelGGL(k_g_div_norm<4>, dim3(blocks), dim3(kBlock), 0, ctx->stream, n, in,
                         A->V.p, w.p, part.p);
    RT_LAUNCH_CHECK();
    RT_CHECK(reduce(1, true, true, column(m)));
    RT_CHECK(ctx->sync_read(column(m), sizeof(double)));
    *norm = ctx->host[0];
    return RT_OK;
  }
  // v_k = w / *norm (device) and z = M^-1 v_k
  int next(int k, const double* norm) {
    hipLaunchKernelGGL(k_g_next, dim3(grid_for(n)), dim3(kBlock), 0, ctx->stream, n, norm, w.p,
                       jacobi(), A->V.p, vec(k), amg ? t.p : z.p);
    RT_LAUNCH_CHECK();
    return amg ? vcycle<double>(ctx, A, t.p, z.p) : RT_OK;
  }
  // iteration k, queued: from z = M^-1 v_k to v_{k+1} and the next z; column k
  // of the Hessenberg matrix (k + 2 values)
  int iterate(int k, bool last) {
    const Level& L = A->levels[0];
    hipStream_t st = ctx->stream;
    const bool pair = pair_serves(L, L.shape64);
    if (pair)
      RT_CHECK((launch_pair<double, PP_PLAIN>(st, L, L.diag64.p, z.p, t.p, nullptr, nullptr,
                                              L.shape64)));
    else
      RT_CHECK((launch_spmv_level<double, SP_PLAIN>(st, L, L.val64.p, L.diag64.p, z.p, nullptr,
                                                    nullptr, t.p, nullptr, nullptr, nullptr,
                                                    L.shape64)));
    const int J = k + 1;
    double* h = column(k);
#define RT_G_DOTS(E_, P_)                                                                        \
  hipLaunchKernelGGL((k_g_dots<E_, P_>), dim3(blocks), dim3(kBlock), 0, st, n, J, L.pair.in(),   \
                     L.pair.sum64.p, t.p, A->V.p, basis.p, w.p, nw, part.p)
#define RT_G_PROJECT(E_, D_)                                                                     \
  hipLaunchKernelGGL((k_g_project<E_, D_>), dim3(blocks), dim3(kBlock), 0, st, n, J, coef.p,     \
                     basis.p, w.p, nw, part.p)
    if (one && pair) RT_G_DOTS(1, true);
    else if (one) RT_G_DOTS(1, false);
    else if (pair) RT_G_DOTS(4, true);
    else RT_G_DOTS(4, false);
    RT_LAUNCH_CHECK();
    RT_CHECK(reduce(J, true, false, h));
    if (one) RT_G_PROJECT(1, true);
    else RT_G_PROJECT(4, true);
    RT_LAUNCH_CHECK();
    RT_CHECK(reduce(J, false, false, h));
    if (one) RT_G_PROJECT(1, false);
    else RT_G_PROJECT(4, false);
    RT_LAUNCH_CHECK();
#undef RT_G_DOTS
#undef RT_G_PROJECT
    RT_CHECK(reduce(1, true, true, h + J));
    return last ? RT_OK : next(k + 1, h + J);
  }
  // t = b - A x
  int residual(const double* b, const double* x) {
    const Level& L = A->levels[0];
    int nbk = 0;
    if (pair_serves(L, L.shape64))
      return pair_resid(ctx, L, x, b, t.p, nullptr, nullptr, A->partA.p, nullptr, &nbk, L.shape64);
    return launch_spmv_level<double, SP_RESID>(ctx->stream, L, L.val64.p, L.diag64.p, x, b, nullptr,
                                               t.p, nullptr, A->partA.p, &nbk, L.shape64);
  }
  // x += M^-1 (V y)
  int correct(int k, const double* y, double* x) {
    GCoef C{};
    for (int j = 0; j < k; ++j) C.c[j] = y[j];
    hipLaunchKernelGGL(k_g_combine, dim3(grid_for(n)), dim3(kBlock), 0, ctx->stream, n, k, C,
                       basis.p, jacobi(), A->V.p, x, t.p);
    RT_LAUNCH_CHECK();
    if (!amg) return RT_OK;
    RT_CHECK(vcycle<double>(ctx, A, t.p, z.p));
    hipLaunchKernelGGL(k_add, dim3(grid_for(n)), dim3(kBlock), 0, ctx->stream, n, z.p, x);
    RT_LAUNCH_CHECK();
    return RT_OK;
  }
};

// Givens rotation zeroing b in (a, b)
void givens(double a, double b, double* c, double* s) {
  if (b == 0.0) {
    *c = 1.0;
    *s = 0.0;
  } else {
    const double r = std::hypot(a, b);
    *c = a / r;
    *s = b / r;
  }
}

int gmres_sorted(rt_ctx* ctx, rt_matrix* A, const double* b, double* x,
                 const rt_gmres_opts* o, rt_solve_stats* stt) {
  hipStream_t st = ctx->stream;
  Gmres G{ctx, A, A->n, o->restart, o->precond == 1 && cycle_depth(A) > 1};
  RT_CHECK(A->partA.reserve(max_partials(A->n)));
  RT_CHECK(G.init());
  if (A->levels[0].pair.on && plain_shape(A->levels[0].shape64)) RT_CHECK(ensure_csr(ctx, A));
  const int64_t n = A->n;
  const int m = G.m;
  // ||c||
  double cnorm = 0.0;
  RT_CHECK(G.div_norm(b, &cnorm));
  if (!std::isfinite(cnorm)) {
    set_error("rt_solve_gmres: right-hand side is not finite");
    return RT_E_ARG;
  }
  if (cnorm == 0.0) {
    hipLaunchKernelGGL(k_fill0, dim3(grid_for(n)), dim3(kBlock), 0, st, n, x);
    RT_LAUNCH_CHECK();
    stt->rel_residual = 0.0;
    return RT_OK;
  }
  const double target = o->tol * cnorm;
  std::vector<double> H((size_t)(m + 1) * m), cs(m), sn(m), g(m + 1), y(m);
  auto Hat = [&](int i, int j) -> double& { return H[(size_t)i * m + j]; };
  int total = 0;
  double beta = 0.0;
  RT_CHECK(G.residual(b, x));
  RT_CHECK(G.div_norm(G.t.p, &beta));
  while (beta > target && total < o->max_iter) {
    if (!std::isfinite(beta)) {
      set_error("rt_solve_gmres: non-finite residual");
      return RT_E_DEVICE;
    }
    RT_CHECK(G.next(0, G.column(m)));
    std::fill(g.begin(), g.end(), 0.0);
    g[0] = beta;
    const int most = std::min(m, o->max_iter - total);   // columns of this cycle
    int k = 0, queued = 0, chunk = 2;
    double est = beta;
    bool stop = false;
    while (k < most && !stop) {
      const int q0 = queued, q1 = std::min(most, queued + chunk);
      for (; queued < q1; ++queued) RT_CHECK(G.iterate(queued, queued + 1 == most));
      RT_CHECK(ctx->sync_read(G.column(q0), sizeof(double) * kGmresCol * (q1 - q0)));
      const double est0 = est;
      const int k0 = k;
      for (; k < q1 && !stop; ++k) {
        const double* h = ctx->host + (size_t)(k - q0) * kGmresCol;
        for (int j = 0; j <= k + 1; ++j) Hat(j, k) = h[j];
        const double hn = h[k + 1];
        // apply the earlier rotations to the new column, then a new one
        for (int j = 0; j < k; ++j) {
          const double a = Hat(j, k), bb = Hat(j + 1, k);
          Hat(j, k) = cs[j] * a + sn[j] * bb;
          Hat(j + 1, k) = -sn[j] * a + cs[j] * bb;
        }
        givens(Hat(k, k), Hat(k + 1, k), &cs[k], &sn[k]);
        Hat(k, k) = cs[k] * Hat(k, k) + sn[k] * Hat(k + 1, k);
        Hat(k + 1, k) = 0.0;
        g[k + 1] = -sn[k] * g[k];
        g[k] = cs[k] * g[k];
        est = std::fabs(g[k + 1]);
        stop = est <= target || hn == 0.0 || !std::isfinite(hn);
      }
      // iterations still needed at the observed rate, three quarters of them,
      // at most as many again as are done
      chunk = 1;
      if (est > 0.0 && est < est0) {
        const double need = std::log(target / est) / (std::log(est / est0) / (k - k0));
        if (std::isfinite(need))
          chunk = (int)std::min<double>(std::max(2, k), std::max(1.0, std::floor(0.75 * need)));
      }
    }
    total += k;
    // y = R^-1 g (upper triangular k x k), x += M^-1 (V y)
    for (int i = k - 1; i >= 0; --i) {
      double s = g[i];
      for (int j = i + 1; j < k; ++j) s -= Hat(i, j) * y[j];
      y[i] = s / Hat(i, i);
    }
    RT_CHECK(G.correct(k, y.data(), x));
    // true residual for the next cycle (and the stopping test)
    RT_CHECK(G.residual(b, x));
    RT_CHECK(G.div_norm(G.t.p, &beta));
  }
  stt->iterations = total;
  stt->rel_residual = beta / cnorm;
  if (!(beta <= target)) {
    set_error("rt_solve_gmres: relative residual %.3e above tolerance %.3e", beta / cnorm,
              o->tol);
    return RT_NOT_CONVERGED;
  }
  return RT_OK;
}

}  // namespace
}  // namespace rt

extern "C" int rt_solve_gmres(rt_ctx* ctx, rt_matrix* A, const double* b, double* x,
                              const rt_gmres_opts* opts, rt_solve_stats* stats) {
  using namespace rt;
  clear_error();
  if (!ctx || !A || !opts || (A->n > 0 && (!b || !x))) {
    set_error("rt_solve_gmres: NULL argument");
    return RT_E_ARG;
  }
  if ((opts->precond != 0 && opts->precond != 1) || !(opts->tol >= 0.0) || opts->max_iter < 0 ||
      opts->restart < 1 || opts->restart > kGmresMaxRestart) {
    set_error("rt_solve_gmres: precond must be 0 or 1, tol >= 0, max_iter >= 0, "
              "1 <= restart <= %d", kGmresMaxRestart);
    return RT_E_ARG;
  }
  RT_CHECK_HIP(hipSetDevice(ctx->device));
  rt::StreamScope release_scope(ctx->stream);   // buffers released here are stream-ordered
  auto t0 = std::chrono::steady_clock::now();
  rt_solve_stats local{};
  rt_solve_stats* stt = stats ? stats : &local;
  *stt = rt_solve_stats{};
  if (A->n == 0) return RT_OK;
  A->resid_ok = false;   // bs, xs and the work vectors are overwritten here
  RT_CHECK(A->xs.reserve(A->n));
  RT_CHECK(A->bs.reserve(A->n));
  RT_CHECK(gather_sorted(ctx, A->nb, A->n, b, A->bs.p));
  RT_CHECK(gather_sorted(ctx, A->nb, A->n, x, A->xs.p));
  const int s = gmres_sorted(ctx, A, A->bs.p, A->xs.p, opts, stt);
  if (s < 0) return s;
  RT_CHECK(scatter_user(ctx, A->nb, A->n, A->xs.p, x));
  RT_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  stt->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return s;
}
