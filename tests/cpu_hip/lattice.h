// A small system for the C++ units of the host emulation: a jittered n x n
// lattice on the unit square through the C ABI.  sign -1: negative masses, so
// negative volumes and a negative definite matrix.
#pragma once
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "rt.h"

struct Lattice {
  int N;
  std::vector<double> pos, h, one, m, e, b, zero;
  rt_step_inputs in{};
  rt_neighbors* nb = nullptr;
  rt_matrix* A = nullptr;

  static rt_amg_opts opts(int levels, int fp32, int tiled) {
    return rt_amg_opts{levels, 16, 0.25, fp32, tiled, RT_SMOOTHER_L1_JACOBI, 2, 1,
                       RT_PROLONG_PIECEWISE};
  }
  Lattice(rt_ctx* ctx, int n, rt_amg_opts o, double sign = 1.0, double support = 1.3)
      : N(n * n), pos(2 * N), h(N, support / n), one(N, 1.0), m(N, sign / N), e(N), b(N),
        zero(N, 0.0) {
    for (int i = 0; i < N; ++i) {
      pos[i] = (i % n + 0.5 + 0.2 * ((i * 7) % 5 - 2) / 5.0) / n;
      pos[N + i] = (i / n + 0.5 + 0.2 * ((i * 3) % 7 - 3) / 7.0) / n;
      e[i] = 1.0 + 0.1 * (i % 11);
      b[i] = (1.0 + (i * 13) % 17) / N;
    }
    in = rt_step_inputs{1e-3, 1.0, 1.0, 0.0, RT_LIMITER_NONE, 2.0, m.data(), one.data(),
                        one.data(), one.data(), zero.data(), e.data(), one.data(), zero.data(),
                        zero.data()};
    if (rt_build_neighbors(ctx, 2, N, N, pos.data(), h.data(), RT_KERNEL_CUBIC_SPLINE, &nb) < 0 ||
        assemble(ctx, o) < 0) {
      printf("FAILED set-up: %s\n", rt_last_error());
      exit(1);
    }
  }
  int assemble(rt_ctx* ctx, rt_amg_opts o) { return rt_assemble(ctx, nb, &in, &o, &A); }
  // its steps of CG from a constant guess (RT_NOT_CONVERGED)
  int steps(rt_ctx* ctx, int precision, int its, std::vector<double>* x) {
    x->assign(N, 0.25);
    rt_solve_opts o{precision, 0, 1e-15, its, 1e-9, 1, 0.0};
    return rt_solve(ctx, A, b.data(), x->data(), &o, nullptr);
  }
  Lattice(const Lattice&) = delete;
  ~Lattice() {
    rt_matrix_free(A);
    rt_neighbors_free(nb);
  }
};
