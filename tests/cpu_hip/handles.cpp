// Handles of matrices in pair form under the host emulation with
// AddressSanitizer, one check per run (argv[1]).
#include <cmath>
#include <cstring>
#include <string>

#include "../../paper_2001_11606_amd/csrc/internal.h"
#include "lattice.h"

namespace {
int failures = 0;
void expect(bool ok, const char* what) {
  printf("%s %s\n", ok ? "ok" : "FAILED", what);
  fflush(stdout);
  failures += !ok;
}
std::vector<double> x;

// a re-assembly whose allocations fail leaves a matrix that can be used
void failed_reassembly(rt_ctx* ctx) {
  Lattice S(ctx, 18, Lattice::opts(1, 0, 1));
  // the step's records are in the cache: the FP32 buffers are what fails
  rt_release_cached(ctx, nullptr);
  expect(S.assemble(ctx, Lattice::opts(1, 0, 1)) == RT_OK, "re-assembly on the kept structure");
  cpuhip_malloc_max = 0;
  expect(S.assemble(ctx, Lattice::opts(1, 1, 1)) == RT_E_OOM, "FP32 copies that do not fit");
  cpuhip_malloc_max = SIZE_MAX;
  expect(S.steps(ctx, RT_PREC_MIXED, 1, &x) == RT_E_STATE, "mixed solve without FP32 copies");
  expect(S.steps(ctx, RT_PREC_FP64, 1, &x) == RT_NOT_CONVERGED, "FP64 solve after it");
  cpuhip_malloc_max = 0;
  expect(S.assemble(ctx, Lattice::opts(8, 0, 1)) == RT_E_OOM, "a hierarchy that does not fit");
  cpuhip_malloc_max = SIZE_MAX;
  expect(S.steps(ctx, RT_PREC_FP64, 1, &x) == RT_NOT_CONVERGED, "FP64 solve after it");
}

// a matrix re-assembled with a hierarchy gives the pair form's memory back
void left_pair_form(rt_ctx* ctx) {
  Lattice S(ctx, 18, Lattice::opts(1, 1, 1));
  auto pair = [&]() -> const rt::PairForm& { return S.A->levels[0].pair; };   // levels may move
  expect(pair().on && pair().col.p && pair().val64.p && pair().val32.p, "assembled in pair form");
  const rt::Level& F = S.A->levels[0];
  expect(!F.rp.p && !F.col.p && !F.val64.p && !F.val32.p, "no buffers of CSR rows");
  expect(S.assemble(ctx, Lattice::opts(8, 1, 1)) == RT_OK && !pair().on, "re-assembled with a hierarchy");
  const rt::PairForm& P = pair();
  expect(!P.col.p && !P.row.p && !P.xcol.p && !P.in_pos.p && !P.val64.p && !P.val32.p && !P.sum64.p,
         "no buffers of the pair form");
  expect(S.steps(ctx, RT_PREC_MIXED, 1, &x) == RT_NOT_CONVERGED, "mixed solve after it");
}

// a matrix in pair form re-assembled untiled is untiled
void left_untiled(rt_ctx* ctx) {
  std::vector<double> want;
  for (int tiled : {1, 0}) {
    Lattice S(ctx, 18, Lattice::opts(1, 1, 1));
    rt_matrix_info info{};
    expect(S.steps(ctx, RT_PREC_FP64, 2, &want) == RT_NOT_CONVERGED, "steps in pair form");
    expect(S.assemble(ctx, Lattice::opts(tiled ? 8 : 1, 1, tiled)) == RT_OK &&
               rt_matrix_get_info(S.A, &info) == RT_OK &&
               (info.level_tile_cols[0] > 0) == (tiled != 0),
           tiled ? "tiled with a hierarchy" : "untiled on request");
    expect(S.steps(ctx, RT_PREC_FP64, 2, &x) == RT_NOT_CONVERGED, "steps after it");
    double d = 0.0, w = 0.0;
    for (int i = 0; i < S.N; ++i) {
      d = std::fmax(d, std::fabs(x[i] - want[i]));
      w = std::fmax(w, std::fabs(want[i]));
    }
    expect(d <= 1e-12 * w, "the same vectors");
  }
}

// an export only reads the matrix
void export_reads(rt_ctx* ctx) {
  Lattice S(ctx, 18, Lattice::opts(1, 1, 1));
  const rt_matrix* A = S.A;
  rt_matrix_info info{};
  rt_matrix_get_info(A, &info);
  std::vector<int64_t> rp[2];
  std::vector<int32_t> col[2];
  std::vector<double> val[2], g[2];
  for (int k = 0; k < 2; ++k) {   // made for the call, then with the level's own rows
    rp[k].resize(S.N + 1);
    col[k].resize(info.nnz);
    val[k].resize(info.nnz);
    g[k].resize(S.N);
    if (k == 1) {
      rt_matrix_set_spmv_shape(S.A, 0, RT_PREC_FP64, 0);
      expect(S.steps(ctx, RT_PREC_FP64, 1, &x) == RT_NOT_CONVERGED && A->levels[0].csr_vals, "a plain shape");
    }
    expect(rt_matrix_export(ctx, A, rp[k].data(), col[k].data(), val[k].data(), g[k].data()) == RT_OK,
           "export");
    if (k == 0)
      expect(!A->levels[0].csr_rows && !A->levels[0].csr_vals && !A->levels[0].rp.p &&
                 !A->levels[0].col.p && !A->levels[0].val64.p,
             "the matrix is as it was");
  }
  expect(rp[0] == rp[1] && col[0] == col[1] && val[0] == val[1] && g[0] == g[1], "the same entries");
}

// a batch only reads its matrices
void batch_reads(rt_ctx* ctx) {
  Lattice P(ctx, 9, Lattice::opts(1, 1, 1)), H(ctx, 7, Lattice::opts(8, 1, 1));
  rt_matrix* mats[] = {P.A, H.A};
  rt_batch* B = nullptr;
  expect(rt_batch_create(ctx, 2, mats, &B) == RT_OK, "a batch of both forms");
  const rt::Level& L = P.A->levels[0];
  expect(L.pair.on && !L.csr_rows && !L.csr_vals && !L.rp.p && !L.col.p && !L.val64.p && !L.val32.p,
         "the matrix in pair form is as it was");
  std::vector<double> b(P.b), got(P.N + H.N, 0.25), want;
  b.insert(b.end(), H.b.begin(), H.b.end());
  rt_solve_opts o{RT_PREC_FP64, 0, 1e-12, 2, 1e-3, 20, 0.0};   // two steps
  expect(rt_batch_solve(ctx, B, b.data(), got.data(), &o, 0, nullptr) == RT_NOT_CONVERGED,
         "batched steps");
  for (Lattice* S : {&P, &H}) {
    x.assign(S->N, 0.25);
    expect(rt_solve(ctx, S->A, S->b.data(), x.data(), &o, nullptr) == RT_NOT_CONVERGED, "its own steps");
    want.insert(want.end(), x.begin(), x.end());
  }
  double d = 0.0, w = 0.0;
  for (size_t i = 0; i < got.size(); ++i) {
    d = std::fmax(d, std::fabs(got[i] - want[i]));
    w = std::fmax(w, std::fabs(want[i]));
  }
  expect(d <= 1e-12 * w, "the same vectors");
  rt_batch_free(B);
}

// the product over several tiles, the last one ragged, against the exported rows:
// the residual of a guess, then three CG steps
void tiles(rt_ctx* ctx) {
  Lattice S(ctx, 24, Lattice::opts(1, 1, 1));
  const rt::PairForm& P = S.A->levels[0].pair;
  expect(P.on && P.ntiles == 3 && S.N % 256 != 0 && P.ext_total > 0, "three tiles");
  rt_matrix_info info{};
  rt_matrix_get_info(S.A, &info);
  std::vector<int64_t> rp(S.N + 1);
  std::vector<int32_t> col(info.nnz);
  std::vector<double> val(info.nnz), g(S.N), diag(S.N), r(S.N), z(S.N), p(S.N), q(S.N), y(S.N);
  expect(rt_matrix_export(ctx, S.A, rp.data(), col.data(), val.data(), g.data()) == RT_OK, "export");
  auto mul = [&](const std::vector<double>& v, std::vector<double>* out) {
    for (int i = 0; i < S.N; ++i) {
      double s = 0.0;
      for (int64_t k = rp[i]; k < rp[i + 1]; ++k) s += val[k] * v[col[k]];
      (*out)[i] = s;
    }
  };
  auto dot = [&](const std::vector<double>& a, const std::vector<double>& b) {
    double s = 0.0;
    for (int i = 0; i < S.N; ++i) s += a[i] * b[i];
    return s;
  };
  for (int i = 0; i < S.N; ++i)
    for (int64_t k = rp[i]; k < rp[i + 1]; ++k)
      if (col[k] == i) diag[i] = val[k];
  for (int its : {0, 3}) {
    x.resize(S.N);
    for (int i = 0; i < S.N; ++i) y[i] = x[i] = 0.5 + 0.01 * ((i * 29) % 41);
    rt_solve_opts o{RT_PREC_FP64, 0, 1e-14, its, 1e-3, 20, 0.0};
    rt_solve_stats st{};
    expect(rt_solve(ctx, S.A, S.b.data(), x.data(), &o, &st) == RT_NOT_CONVERGED && st.iterations == its,
           its ? "three steps" : "no step");
    mul(y, &q);
    for (int i = 0; i < S.N; ++i) {
      r[i] = S.b[i] - q[i];
      p[i] = z[i] = r[i] / diag[i];
    }
    double rz = dot(r, z);
    for (int k = 0; k < its; ++k) {
      mul(p, &q);
      const double alpha = rz / dot(p, q);
      for (int i = 0; i < S.N; ++i) {
        y[i] += alpha * p[i];
        r[i] -= alpha * q[i];
        z[i] = r[i] / diag[i];
      }
      const double next = dot(r, z);
      for (int i = 0; i < S.N; ++i) p[i] = z[i] + next / rz * p[i];
      rz = next;
    }
    const double rel = std::sqrt(dot(r, r) / dot(S.b, S.b));
    double d = 0.0, w = 0.0;
    for (int i = 0; i < S.N; ++i) {
      d = std::fmax(d, std::fabs(x[i] - y[i]));
      w = std::fmax(w, std::fabs(y[i]));
    }
    // rounding of sums of some 30 terms, three times
    expect(std::fabs(st.rel_residual - rel) <= 1e-11 * rel && d <= 1e-11 * w, "the host's values");
  }
}
}  // namespace

int main(int argc, char** argv) {
  rt_ctx* ctx = nullptr;
  if (argc < 2 || rt_create(&ctx, 0, nullptr) < 0) return 1;
  const std::string what = argv[1];
  if (what == "failed_reassembly") failed_reassembly(ctx);
  else if (what == "left_pair_form") left_pair_form(ctx);
  else if (what == "left_untiled") left_untiled(ctx);
  else if (what == "export_reads") export_reads(ctx);
  else if (what == "batch_reads") batch_reads(ctx);
  else if (what == "tiles") tiles(ctx);
  else return 1;
  rt_destroy(ctx);
  printf(failures ? "%d failures\n" : "all ok\n", failures);
  return failures ? 1 : 0;
}
