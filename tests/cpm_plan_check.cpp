// Walks the launch plan of the matrix-core nnCP kernel (cpm_plan.h) as the kernel's waves do, for every
// shape and thread count that it takes, and counts how often each unit (16-row tile and range of the
// contracted index) of the two products comes up: exactly once, within the registers of the variant.  The
// partial sums of the updates stay within their LDS.
// Prints the number of plans and the first shapes that fail; the exit status is 1 if any does.
// With arguments (rank, threads, modes): whether the kernel is the one that such a fit goes to.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "cpm_plan.h"

using namespace nnc;

template <int NS>
static bool once(const CpmProd &p, int ks, int nw, int nr) {
  std::vector<int> seen(p.tiles * p.split, 0);
  if (4LL * p.kper * p.split < ks || 4LL * p.kper * (p.split - 1) >= ks) return false;  // no range empty, none missing
  if (nr && (p.passes != 1 || (p.kper + 3) / 4 * 4 * NS > nr)) return false;
  for (int pass = 0; pass < p.passes; ++pass)
    for (int w = 0; w < nw; ++w) {
      // a wave's units after its first are reached only if the first is one
      if (cpm_unit<NS>(p, w, nw, pass, 0).q >= p.split) continue;
      for (int s = 0; s < NS; ++s) {
        const CpmUnit u = cpm_unit<NS>(p, w, nw, pass, s);
        if (u.q < p.split) ++seen.at(u.t + p.tiles * u.q);
      }
    }
  for (int n : seen)
    if (n != 1) return false;
  return true;
}

// The partial sums of every M_n, for every rank of a fit, stay within their region of the LDS.
static bool sums_fit(const CpmArgs &a, int threads) {
  const int nw = threads / 64;
  for (int RS : {8, 16, 32})
    for (int nq = 1; 4 * nq <= RS; ++nq)
      for (int n = 0; n < a.d; ++n) {
        const int group = n < a.s ? a.pL : a.pR;
        if ((n < a.s ? a.s : a.d - a.s) == 1) continue;
        const int In = a.dims[n], per = 64 * std::max(nw - 2, 1) / (In * nq);
        if ((int64_t)In * cpm_sum_ranges(per, group / In) * 4 * nq > std::max(4 * threads, a.maxdim * RS)) return false;
      }
  return true;
}

static bool plan_ok(int d, const int64_t *dims, int threads) {
  const CpmPlan pl = cpm_plan(d, dims, threads);
  const CpmArgs &a = pl.a;
  const int nw = threads / 64;
  const bool v = pl.ns == 8   ? pl.nr == 64 && once<8>(a.v, a.pR, nw, pl.nr)
                 : pl.ns == 4 ? once<4>(a.v, a.pR, nw, pl.nr)
                              : pl.ns == 1 && once<1>(a.v, a.pR, nw, pl.nr);
  return v && once<1>(a.u, a.pL, nw, pl.nr) && sums_fit(a, threads);
}

int main(int argc, char **argv) {
  if (argc > 3) {
    int64_t dims[8], size = 1;
    for (int k = 3; k < argc; ++k) size *= dims[k - 3] = atoi(argv[k]);
    printf("%d\n", cpm_fits(argc - 3, dims, size, atoi(argv[1]), atoi(argv[2])));
    return 0;
  }
  long plans = 0, bad = 0, streamed_ranges = 0;
  for (int d = 3; d <= 5; ++d) {
    // the plan depends on the two groups' products alone (and the largest mode): one shape for each pair
    std::set<std::pair<int, int>> pairs;
    auto group = [](int n) {
      std::set<std::vector<int>> out;
      std::set<int> prod;
      for (int x = 1; x <= 64; ++x)
        for (int y = 1; y <= (n > 1 ? 64 : 1); ++y)
          for (int z = 1; z <= (n > 2 ? 64 : 1); ++z)
            if (prod.insert(x * y * z).second) out.insert(n == 1 ? std::vector<int>{x} : n == 2 ? std::vector<int>{x, y} : std::vector<int>{x, y, z});
      return out;
    };
    const auto left = group((d + 1) / 2), right = group(d / 2);
    for (const auto &l : left)
      for (const auto &r : right) {
        int64_t dims[5], size = 1;
        int n = 0;
        for (int x : l) dims[n++] = x;
        for (int x : r) dims[n++] = x;
        for (int k = 0; k < d; ++k) size *= dims[k];
        if (size < 512 || size > (1 << 17)) continue;
        for (int threads = 64; threads <= kCpmMaxThreads; threads += 64) {
          if (!cpm_takes(d, dims, size, 1, threads)) continue;
          ++plans;
          const CpmPlan pl = cpm_plan(d, dims, threads);
          streamed_ranges += !pl.nr && pl.a.v.split > 1;
          if (plan_ok(d, dims, threads)) continue;
          if (++bad > 10) continue;
          printf("bad:");
          for (int k = 0; k < d; ++k) printf(" %d", (int)dims[k]);
          printf(" threads %d ns %d nr %d split %d\n", threads, pl.ns, pl.nr, pl.a.v.split);
        }
      }
  }
  printf("%ld plans, %ld streamed in ranges, %ld bad\n", plans, streamed_ranges, bad);
  return bad || !streamed_ranges;
}
