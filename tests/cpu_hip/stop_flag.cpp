// The stop flag of the PCG loop, under the host emulation with AddressSanitizer.
//
// 1. k_pupdate at the end of a loop and k_update at a breakdown, with blocks
//    that start while block 0 ends (cpuhip::LateWrite): no row may change, whatever
//    the waves of such a block find in the flag and in LDS.
// 2. Whole solves that end in either way (a matrix of negative volumes has
//    p.Ap < 0), FP64 and mixed, plain and with late blocks: the same solution, bit
//    for bit; printed, so that builds with other reductions can be compared.
#include "../../paper_2001_11606_amd/csrc/solve.hip"
#include "lattice.h"

namespace {
using namespace rt;

int failures = 0;
void expect(bool ok, const char* what) {
  printf("%s %s\n", ok ? "ok" : "FAILED", what);
  fflush(stdout);
  failures += !ok;
}

struct Loop {   // the vectors and scalars of one loop of n rows
  int n, np;
  std::vector<double> x, r, p, q, dinv, pa, pb, pq, partA, partB, s;
  int32_t stop[STOP_WORDS] = {0, 0};
  Loop(int rows, int parts, double a, double b, double dot)
      : n(rows), np(parts), x(rows, 2.0), r(rows, 3.0), p(rows, 5.0), q(rows, 7.0),
        dinv(rows, 0.5), pa(parts, a), pb(parts, b), pq(parts, dot), partA(rows), partB(rows),
        s(S_COUNT, 0.0) {
    s[S_RZ] = 1.0;
    s[S_THR] = 1e-3;
    s[S_CWTHR] = INFINITY;
  }
  int blocks() const { return vec_blocks(n); }
  void pupdate() {
    hipLaunchKernelGGL((k_pupdate<double, true, 1>), dim3(blocks()), dim3(kBlock), 0, nullptr,
                       (int64_t)n, np, (const double*)pa.data(), (const double*)pb.data(),
                       (const double*)nullptr, 0, s.data(), (const double*)r.data(),
                       (const double*)dinv.data(), (const double*)nullptr, p.data(), stop);
  }
  void update() {
    hipLaunchKernelGGL((k_update<double, true, CW_NONE, false, 1>), dim3(blocks()), dim3(kBlock), 0,
                       nullptr, (int64_t)n, PairIn{}, (const double*)nullptr, np,
                       (const double*)pq.data(), 0, s.data(), x.data(), r.data(),
                       (const double*)p.data(), (const double*)q.data(),
                       (const double*)dinv.data(), (const double*)nullptr, partA.data(),
                       partB.data(), (double*)nullptr, stop);
  }
};
bool all(const std::vector<double>& v, double want) {
  return std::all_of(v.begin(), v.end(), [=](double e) { return e == want; });
}

void late_kernels() {
  Loop other(256, 600, 1.0, 1.0, 1.0);   // a loop that goes on: what it leaves in LDS
  {
    Loop l(1024, 600, 1e-9, 1.0, 1.0);   // ||r||^2 below the threshold
    cpuhip::LateWrite late{l.stop, STOP_WORDS, [&] { other.pupdate(); }};
    cpuhip::g_late = &late;
    l.pupdate();
    cpuhip::g_late = nullptr;
    expect(all(l.p, 5.0) && l.s[S_STOP] == 1.0, "p update at the end of a loop, late blocks");
    l.update();   // the next launches leave everything as it is
    l.pupdate();
    expect(all(l.x, 2.0) && all(l.r, 3.0) && all(l.p, 5.0) && l.s[S_ITS] == 1.0,
           "iteration after the end of a loop");
  }
  {
    Loop l(1024, 600, 1.0, 1.0, -1.0);   // p.Ap negative
    cpuhip::LateWrite late{l.stop, STOP_WORDS, [&] { other.update(); }};
    cpuhip::g_late = &late;
    l.update();
    cpuhip::g_late = nullptr;
    expect(all(l.x, 2.0) && all(l.r, 3.0) && l.s[S_BAD] == 1.0, "x, r update at a breakdown, late blocks");
    l.pupdate();
    l.update();
    expect(all(l.x, 2.0) && all(l.p, 5.0) && l.s[S_ITS] == 0.0, "launches after a breakdown");
  }
}

void solves(rt_ctx* ctx) {
  for (double sign : {1.0, -1.0}) {
    Lattice S(ctx, 18, Lattice::opts(1, 1, 1), sign);
    const int N = S.N;
    for (int mixed = 0; mixed < 2; ++mixed) {
      std::vector<double> got[2];
      rt_solve_stats st[2];
      int status[2];
      cpuhip::LateWrite late{};
      for (int k = 0; k < 2; ++k) {   // the work buffers exist after the first
        got[k].assign(N, 0.25);
        if (k == 1) {
          late.words = S.A->stop.p;
          late.n = STOP_WORDS;
          cpuhip::g_late = &late;
        }
        rt_solve_opts o{mixed ? RT_PREC_MIXED : RT_PREC_FP64, 0, 1e-6, 200, 1e-3, 20, 0.0};
        status[k] = rt_solve(ctx, S.A, S.b.data(), got[k].data(), &o, &st[k]);
        cpuhip::g_late = nullptr;
      }
      uint64_t hash = 1469598103934665603ull;
      for (double v : got[0]) {
        uint64_t bits;
        memcpy(&bits, &v, 8);
        hash = (hash ^ bits) * 1099511628211ull;
      }
      printf("solve sign=%g mixed=%d status=%d iterations=%d x=%016llx\n", sign, mixed, status[0],
             st[0].iterations, (unsigned long long)hash);
      if (sign > 0) expect(status[0] == RT_OK && st[0].iterations > 3, "a solve that converges");
      else
        expect(status[0] == RT_NOT_CONVERGED && st[0].iterations == 0 && all(got[0], 0.25),
               "a solve that breaks down leaves x");
      expect(status[0] == status[1] && st[0].iterations == st[1].iterations &&
                 !memcmp(got[0].data(), got[1].data(), 8 * N),
             "the same bits with late blocks");
    }
  }
}

}  // namespace

int main() {
  late_kernels();
  rt_ctx* ctx = nullptr;
  if (rt_create(&ctx, 0, nullptr) < 0) return 1;
  solves(ctx);
  rt_destroy(ctx);
  printf(failures ? "%d failures\n" : "all ok\n", failures);
  return failures ? 1 : 0;
}
