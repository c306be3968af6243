// The launch plan of the matrix-core nnCP kernel (cpm_kernels.hip): how the two products of a sweep
// are divided over a workgroup's waves, which variant of the kernel runs, and its LDS.  Nothing here
// needs a GPU; a host compiler takes it as well.
#pragma once
#include <stdint.h>
#include <string.h>

#include <algorithm>

#ifdef __HIPCC__
#define NNC_HD __host__ __device__
#else
#define NNC_HD
#endif

namespace nnc {

constexpr int kCpmWaves = 8;      // two per SIMD, 256 registers each
constexpr int kCpmMaxThreads = 64 * kCpmWaves;
constexpr int64_t kCpmLds = 158 * 1024;

// One of the two products: `tiles` 16-row tiles times `split` ranges of `kper` steps (a step is
// four values of the contracted index) are units, unit u = tile + tiles * range; wave w takes
// units w, w + waves, ..., NS at a time (NS > 1 only without ranges: those tiles share their
// operand rows), in `passes` passes.
struct CpmProd {
  int tiles, split, kper, passes;
};

struct CpmArgs {
  int d, s;
  int dims[5];
  int size, pL, pR, sumdim, maxdim;  // sumdim: modes rounded up to 4 rows
  CpmProd v, u;
};

// The unit of one wave at slot s of a pass: tile t, range q (q >= split: none).
struct CpmUnit {
  int t, q;
};
template <int NS>
NNC_HD inline CpmUnit cpm_unit(const CpmProd &p, int wave, int nw, int pass, int s) {
  CpmUnit u{wave + nw * (NS * pass + s), 0};
  if (NS == 1) {
    while (u.t >= p.tiles) {
      u.t -= p.tiles;
      ++u.q;
    }
  } else if (u.t >= p.tiles) {
    u.q = p.split;
  }
  return u;
}

// The plan: V's tiles go `ns` at a time, U's one at a time; a lane keeps `nr` values of T for each
// product in registers, or (nr = 0) reads them from the L2 each sweep.
struct CpmPlan {
  CpmArgs a;
  int ns, nr;
};

inline CpmProd cpm_prod(int rows, int ks, int nw, int ns) {
  CpmProd p;
  p.tiles = (rows + 15) / 16;
  const int steps = (ks + 3) / 4;
  p.split = ns > 1 ? 1 : std::max(1, std::min(nw / p.tiles, steps));
  p.kper = (steps + p.split - 1) / p.split;
  p.split = (steps + p.kper - 1) / p.kper;
  p.passes = (p.tiles * p.split + nw * ns - 1) / (nw * ns);
  return p;
}

// Values of T that a lane holds for a product.
inline int cpm_regs(const CpmProd &p, int ns) { return p.passes * ((p.kper + 3) / 4) * 4 * ns; }

inline CpmPlan cpm_plan(int d, const int64_t *dims, int threads) {
  CpmPlan pl;
  CpmArgs &a = pl.a;
  memset(&a, 0, sizeof a);
  a.d = d;
  a.s = (d + 1) / 2;
  a.pL = a.pR = 1;
  for (int k = 0; k < d; ++k) {
    a.dims[k] = (int)dims[k];
    (k < a.s ? a.pL : a.pR) *= a.dims[k];
    a.sumdim += (a.dims[k] + 3) & ~3;
    a.maxdim = std::max(a.maxdim, a.dims[k]);
  }
  a.size = a.pL * a.pR;
  // V's tiles: several share their operand rows once every wave has some; fewer than the waves are
  // split into ranges of the contracted index instead
  const int nw = threads / 64, per = ((a.pL + 15) / 16 + nw - 1) / nw;
  pl.ns = per > 4 ? 8 : (per > 1 ? 4 : 1);
  a.v = cpm_prod(a.pL, a.pR, nw, pl.ns);
  a.u = cpm_prod(a.pR, a.pL, nw, 1);
  // T in registers when each product takes one pass and a lane's share fits 32 or 64 values per
  // layout, else from the L2 each sweep, by one slot (with V's ranges) or by four
  const int g = std::max(cpm_regs(a.v, pl.ns), cpm_regs(a.u, 1));
  pl.nr = g > 64 || a.v.passes > 1 || a.u.passes > 1 ? 0 : (g > 32 || pl.ns == 8 ? 64 : 32);
  if (!pl.nr && pl.ns > 1) {
    pl.ns = 4;
    a.v = cpm_prod(a.pL, a.pR, nw, pl.ns);
  }
  return pl;
}

// Rows of every array over ranks hold RS = 8, 16 or 32 values, zeros past the rank.  LDS floats of
// a fit with `threads` threads:
//   factors, two buffers | Grams (d RS WS) | H (RS WS) | partial sums of M_n (cpm_sum_ranges times In
//   rows of the fit's quads; or, with one mode in a group, none) | KR of the left group | KR of the right group (groups of one mode are the
//   factor itself) | V or U, by ranges of the contracted index.  The residual's FP64 sums reuse
//   V and U, which are at least 4 floats a thread.
// Rows of the Grams and of H are WS = RS + 4 floats apart: an update reads 16 of them at once, 16
// bytes each, from 64 different banks.  All of it starts as zeros: operand reads past an array's
// last row meet zeros of T, and have to be finite.
// The ranges that M_n's sum over `terms` terms is split into, by the fit's own rank (nq quads) alone: the
// threads of the waves but the two with a Gram and H to form, each with a quad of a row.  In times the
// ranges is at most 64 max(nw - 2, 1) / nq, or In where that is less than one range: at most 4 * threads
// or maxdim * RS floats of sums.
NNC_HD inline int cpm_sum_ranges(int per, int terms) {
  const int most = terms < 16 ? terms : 16, n = per < most ? per : most;
  return n > 1 ? n : 1;
}

inline int cpm_rs(int r) { return r <= 8 ? 8 : (r <= 16 ? 16 : 32); }

inline int64_t cpm_lds_floats(const CpmArgs &a, int RS, int threads) {
  int64_t n = 2 * a.sumdim * RS + (int64_t)(a.d + 1) * RS * (RS + 4);
  n += std::max<int64_t>(4 * (int64_t)threads, (int64_t)a.maxdim * RS);
  if (a.s > 1) n += a.pL * RS;
  if (a.d - a.s > 1) n += a.pR * RS;
  n += std::max<int64_t>(std::max<int64_t>((int64_t)a.v.split * a.pL, (int64_t)a.u.split * a.pR) * RS, 4 * (int64_t)threads);
  return n + 128 * RS;  // products of one pass read up to 32 step groups of rows
}

// Cores of fewer than 512 entries stay with nncp_k: there is little to gain there (4.6 us a sweep
// of 3 x 4 x 5 at rank 5 against 3.1 here), and such small fits carry every change of rounding far
// (an order of sums of its own moved single factors 2e-6, as far as either lies from 64 bits).
// Orders 3 to 5 with modes of at most 64 (one wave forms a Gram, one pass of the block an
// update) whose working set fits one CU; other shapes stay with nncp_k.
inline bool cpm_takes(int d, const int64_t *dims, int64_t size, int max_rank, int threads) {
  if (d < 3 || d > 5 || size < 512 || size > (1 << 17) || max_rank > 32) return false;
  for (int k = 0; k < d; ++k)
    if (dims[k] > 64) return false;
  threads = std::min(threads, kCpmMaxThreads);
  return cpm_lds_floats(cpm_plan(d, dims, threads).a, cpm_rs(max_rank), threads) * 4 <= kCpmLds;
}

// Of those, the shapes that nncp_k is sooner with (us a sweep, here and there; 1710 fits of 3 to 5 modes):
//   - 3-way tensors read from the L2 here at ranks up to 10, whose products fill at most 10 of 16 columns:
//     nncp_k has one contraction to do for them too (40 x 40 x 40 at rank 3 43 and 19, 33 x 33 x 33 at
//     8 36 and 19; 21 x 38 x 61 at 16 27 and 32);
//   - small 3-way tensors at ranks 17 .. 22, held as 32 here (9 x 8 x 8 at 17 7.8 and 6.6, 7 x 13 x 13 at
//     18 8.4 and 8.0; over 1400 entries 3 % sooner here and more);
//   - 4-way tensors of a few rows and a long right group, whose two modes share the work of a rank here,
//     while nncp_k holds the tensor in its LDS (2 x 1 x 51 x 39 at rank 8 33 and 18, 7 x 2 x 53 x 38 at 3
//     34 and 25; 4 x 8 x 12 x 16 at 10 9.2 and 24).  The line is a fit: no shape beyond it lost more than
//     a quarter, one before it is 14 % slower.
inline bool cpm_later(const CpmPlan &pl, int max_rank) {
  const CpmArgs &a = pl.a;
  if (a.d == 3) return (!pl.nr && max_rank <= 10) || (max_rank > 16 && max_rank <= 22 && a.size <= 1400);
  const int64_t quads = (max_rank + 3) / 4 * 4;
  return a.d == 4 && !pl.nr && pl.ns == 1 && a.size <= 36000 && (int64_t)a.pR * a.pR > 6400 * a.pL * quads;
}

inline bool cpm_fits(int d, const int64_t *dims, int64_t size, int max_rank, int threads) {
  return cpm_takes(d, dims, size, max_rank, threads) &&
         !cpm_later(cpm_plan(d, dims, std::min(threads, kCpmMaxThreads)), max_rank);
}

}  // namespace nnc
