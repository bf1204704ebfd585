// Offsets of the tiles' external columns (k_pair_scan) under the host emulation:
// a sum past 2^31 arrives whole, so that the pair form can be given up for it.
#include "../../paper_2001_11606_amd/csrc/pair.hip"

int main() {
  using namespace rt;
  int failures = 0;
  for (const int64_t nt : {(int64_t)1, (int64_t)1500, ((int64_t)1 << 20) + 77}) {
    std::vector<PairStat> stat(nt, PairStat{kPairMaxExt, 2500, 90, 0, 4000});
    stat[nt / 2].ext = 11;
    std::vector<int64_t> xoff(nt + 1, -1);
    PairTotals t{};
    hipLaunchKernelGGL(k_pair_scan, dim3(1), dim3(kScanThreads), 0, nullptr, nt,
                       (const PairStat*)stat.data(), xoff.data(), &t);
    int64_t o = 0;
    bool ok = true;
    for (int64_t k = 0; k < nt; ++k) {
      ok = ok && xoff[k] == o;
      o += stat[k].ext;
    }
    ok = ok && xoff[nt] == o && t.ext == o && t.distinct == 2500 * nt && t.nnz == 4000 * nt &&
         t.max_ext == (nt > 1 ? kPairMaxExt : 11) && t.bad == 0;
    printf("%s %lld tiles, %lld external columns, %lld found\n", ok ? "ok" : "FAILED", (long long)nt,
           (long long)o, (long long)t.ext);
    failures += !ok;
  }
  printf(failures ? "%d failures\n" : "all ok\n", failures);
  return failures ? 1 : 0;
}
