// A plain shape requested of a batch in pair form runs on CSR rows made from the
// pairs: the rows and the solution against those of the matrices, under the
// host emulation with AddressSanitizer.
#include <algorithm>

#include "../../paper_2001_11606_amd/csrc/batch.hip"
#include "lattice.h"

namespace {
int failures = 0;
void expect(bool ok, const char* what) {
  printf("%s %s\n", ok ? "ok" : "FAILED", what);
  fflush(stdout);
  failures += !ok;
}
}  // namespace

int main() {
  rt_ctx* ctx = nullptr;
  if (rt_create(&ctx, 0, nullptr) < 0) return 1;
  {
    Lattice P(ctx, 17, Lattice::opts(1, 1, 1)), Q(ctx, 6, Lattice::opts(1, 1, 1));
    Lattice* sys[] = {&P, &Q};
    rt_matrix* mats[] = {P.A, Q.A};
    rt_batch* B = nullptr;
    expect(rt_batch_create(ctx, 2, mats, &B) == RT_OK && B->L.pair.on && !B->L.csr_vals,
           "a batch in pair form");
    std::vector<double> b(P.b), first(P.N + Q.N), got(P.N + Q.N);
    b.insert(b.end(), Q.b.begin(), Q.b.end());
    auto solve = [&](int prec, std::vector<double>* x) {
      rt_solve_opts o{prec, 0, 1e-12, 1, 1e-3, 1, 0.0};   // one step, replayed
      x->assign(b.size(), 0.25);
      return rt_batch_solve(ctx, B, b.data(), x->data(), &o, 1, nullptr);
    };
    auto near = [&](const std::vector<double>& x, const std::vector<double>& y, double bar) {
      double d = 0.0, w = 0.0;
      for (size_t i = 0; i < x.size(); ++i) {
        d = std::max(d, std::fabs(x[i] - y[i]));
        w = std::max(w, std::fabs(y[i]));
      }
      return d <= bar * w;
    };
    expect(solve(RT_PREC_FP64, &first) == RT_NOT_CONVERGED && !B->L.csr_vals, "steps in pair form");
    rt_batch_set_spmv_shape(B, RT_PREC_FP64, 1);
    expect(solve(RT_PREC_FP64, &got) == RT_NOT_CONVERGED && B->L.csr_vals &&
               !rt::pair_serves(B->L, 1),
           "the plain shape runs on CSR rows");
    expect(near(got, first, 1e-12), "the same vectors");
    // the rows of both problems: those the matrices make from their lists
    for (int p = 0; p < 2; ++p) {
      expect(rt::ensure_csr(ctx, sys[p]->A) == RT_OK, "the matrix's own rows");
      const rt::Level &L = B->L, &M = sys[p]->A->levels[0];
      const int64_t r0 = B->row_off[p];
      bool same = true;
      for (int64_t i = 0; i < M.n; ++i) {
        const int64_t a = L.rp.p[r0 + i], m = M.rp.p[i + 1] - M.rp.p[i];
        same = same && L.rp.p[r0 + i + 1] - a == m;
        // the lists' order of cells against ascending columns
        std::vector<std::pair<int64_t, int64_t>> at;
        for (int64_t q = M.rp.p[i]; q < M.rp.p[i + 1]; ++q) at.emplace_back(r0 + M.col.p[q], q);
        std::sort(at.begin(), at.end());
        for (int64_t k = 0; same && k < m; ++k)
          same = L.col.p[a + k] == at[k].first && L.val64.p[a + k] == M.val64.p[at[k].second] &&
                 L.val32.p[a + k] == M.val32.p[at[k].second];
      }
      for (int64_t i = r0 + M.n; i < B->row_off[p + 1]; ++i)   // padding
        same = same && L.rp.p[i] == L.rp.p[i + 1];
      expect(same, "the same rows");
    }
    rt_batch_set_spmv_shape(B, RT_PREC_MIXED, 1);
    expect(solve(RT_PREC_MIXED, &got) == RT_NOT_CONVERGED && near(got, first, 1e-5),
           "mixed on the rows");
    rt_batch_set_spmv_shape(B, RT_PREC_FP64, -1);
    expect(solve(RT_PREC_FP64, &got) == RT_NOT_CONVERGED && got == first,
           "pair form again, the same bits");
    rt_batch_free(B);
  }
  {   // a re-assembly makes the rows of a plain shape set before it
    Lattice P(ctx, 9, Lattice::opts(1, 1, 1));
    std::vector<double> x(P.N, 0.25), own;
    rt_matrix_set_spmv_shape(P.A, 0, RT_PREC_FP64, 1);
    expect(!P.A->levels[0].csr_vals && P.assemble(ctx, Lattice::opts(1, 1, 1)) == RT_OK &&
               P.A->levels[0].csr_vals,
           "rows after a re-assembly");
    own.assign(P.N, 0.25);
    rt_solve_opts o{RT_PREC_FP64, 0, 1e-12, 2, 1e-3, 20, 0.0};
    expect(rt_solve_noalloc(ctx, P.A, P.b.data(), x.data(), &o, nullptr) == RT_NOT_CONVERGED &&
               rt_solve(ctx, P.A, P.b.data(), own.data(), &o, nullptr) == RT_NOT_CONVERGED && x == own,
           "rt_solve_noalloc runs the shape");
  }
  rt_destroy(ctx);
  printf(failures ? "%d failures\n" : "all ok\n", failures);
  return failures ? 1 : 0;
}
