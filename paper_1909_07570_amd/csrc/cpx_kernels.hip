// Small steps of the nonnegative CP fit of the data tensor itself (the nnCPD step of
// Algorithm 2), around the two X-streaming contractions it shares with the Tucker sweep.
//
// With Z = X x_{d-1} B_{d-1}^T (rank index last) and T = X x_0 B_0^T (rank index first), the
// MTTKRP of every mode is a rank-wise ("diagonal") contraction of Z or T with the current
// factors of the remaining modes:
//   M_n[i][rho] = sum_{a, c} Y[a][i][c][rho] WA[a][rho] WC[c][rho]      (rank index last)
//   M_n[i][rho] = sum_{a, c} Y[rho][a][i][c] WA[a][rho] WC[c][rho]      (rank index first)
// where a runs over the modes of Y before mode n and c over those after it, and WA / WC are
// the Khatri-Rao rows of those modes' factors.  The multiplicative update then uses
// H_n = Hadamard product of the other factors' Grams (reading R1 applied to CP).
#include <string.h>

#include <algorithm>
#include <mutex>
#include <set>

#include "nnc_internal.h"

namespace nnc {

constexpr int kDiagThreads = 256;

struct DiagArgs {
  const float *Y;
  const float *WA, *WC;  // null: weight 1
  int64_t A, Nt, C;
  int r;
  int rho_first;
  float *out;  // [slices][Nt][r]
  int slices;
  // block 0 of the kernels with a Gram (GRAM) forms gS = gB^T gB (gN x r) of another factor
  const float *gB;
  float *gS;
  int gN;
};

constexpr int kGramSums = 1024;  // partial sums of a Gram: 1024 / r^2 row sets times its entries

// S = B^T B (N x r, r <= 16 TR) by a block of kDiagThreads threads with the sums of gram_block_k, bit for
// bit: entry e of row set k (rows j with j mod sets == k, ascending) is one FP32 accumulator, whose
// 16 x 16 x 4 MFMA adds four rows one after the other, and the sets are added in order.  NB sets of a
// wave run side by side; a lane's row of a step is both operands.
template <int TR>
static __device__ inline void gram_sets(const float *__restrict__ B, int N, int r, float *__restrict__ S, float *part) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int kW = kDiagThreads / 64, NB = 4;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rr = r * r, sets = kGramSums / rr;
  const int steps = ((N + sets - 1) / sets + 3) / 4;
  for (int k0 = wave; k0 < sets; k0 += NB * kW) {
    f4 acc[NB][TR][TR];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int p = 0; p < TR; ++p)
#pragma unroll
        for (int q = 0; q < TR; ++q) acc[n][p][q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = 0; s < steps; ++s) {
      float x[NB][TR];
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int row = k0 + n * kW + (4 * s + lg) * sets;  // sets past the last are not stored
#pragma unroll
        for (int p = 0; p < TR; ++p) {
          const float v = B[min(row, N - 1) * r + min(16 * p + li, r - 1)];
          x[n][p] = row < N ? v : 0.f;
        }
      }
#pragma unroll
      for (int p = 0; p < TR; ++p)
#pragma unroll
        for (int q = 0; q < TR; ++q)
#pragma unroll
          for (int n = 0; n < NB; ++n)
            acc[n][p][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[n][p], x[n][q], acc[n][p][q], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int p = 0; p < TR; ++p)
#pragma unroll
        for (int q = 0; q < TR; ++q)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int a = 16 * p + 4 * lg + j, b = 16 * q + li, k = k0 + n * kW;
            if (a < r && b < r && k < sets) part[k * rr + a * r + b] = acc[n][p][q][j];
          }
  }
  __syncthreads();
  for (int e = tid; e < rr; e += kDiagThreads) {
    float t = part[e];
    for (int k = 1; k < sets; ++k) t += part[k * rr + e];
    S[e] = t;
  }
}

// Block 0 of a launch with a Gram: true where the caller is done.  part: the block's LDS, at least
// kGramSums floats.
template <int RM>
static __device__ inline bool diag_gram(const DiagArgs &g, float *part) {
  static_assert(kDiagThreads * RM >= kGramSums, "the Gram's sums fit the block's LDS");
  if (blockIdx.x) return false;
  gram_sets<(RM + 15) / 16>(g.gB, g.gN, g.r, g.gS, part);
  return true;
}

static __device__ inline float diag_y(const DiagArgs &g, int64_t a, int64_t i, int64_t c, int rho) {
  const int64_t e = (a * g.Nt + i) * g.C + c;
  return g.rho_first ? g.Y[(int64_t)rho * g.A * g.Nt * g.C + e] : g.Y[e * g.r + rho];
}

static __device__ inline float diag_w(const DiagArgs &g, int64_t a, int64_t c, int rho) {
  float w = g.WA ? g.WA[a * g.r + rho] : 1.f;
  if (g.WC) w *= g.WC[c * g.r + rho];
  return w;
}

// C > 1: block (i, slice); the threads stride over the flattened (a, c) range of the slice
// (c fastest, contiguous in Y) and the partial sums are combined by a fixed pairwise tree
// (thread t adds thread t + h for h = 128, 64, ..., 1).  The tree's two cross-wave steps
// go through LDS; its steps inside wave 0 are shuffles that pair the same lanes.
template <int RM, bool GRAM>
__global__ __launch_bounds__(kDiagThreads) void diag_inner_k(DiagArgs g) {
  static_assert(kDiagThreads == 256, "the tree below has two cross-wave steps");
  __shared__ float red[kDiagThreads * RM];
  if constexpr (GRAM)
    if (diag_gram<RM>(g, red)) return;
  const int t = threadIdx.x, block = blockIdx.x - (GRAM ? 1 : 0);
  const int64_t i = block % g.Nt;
  const int s = (int)(block / g.Nt);
  const int64_t F = g.A * g.C;
  const int64_t f0 = F * s / g.slices, f1 = F * (s + 1) / g.slices;
  float acc[RM];
#pragma unroll
  for (int q = 0; q < RM; ++q) acc[q] = 0.f;
  int64_t f = f0 + t;
  int64_t a = f / g.C, c = f - a * g.C;  // advanced incrementally below
  for (; f < f1; f += kDiagThreads) {
#pragma unroll
    for (int q = 0; q < RM; ++q)
      if (q < g.r) acc[q] = fmaf(diag_y(g, a, i, c, q), diag_w(g, a, c, q), acc[q]);
    c += kDiagThreads;
    if (c >= g.C) {
      a += c / g.C;
      c %= g.C;
    }
  }
#pragma unroll
  for (int q = 0; q < RM; ++q) red[q * kDiagThreads + t] = acc[q];
  __syncthreads();
  if (t < 128)
#pragma unroll
    for (int q = 0; q < RM; ++q) red[q * kDiagThreads + t] += red[q * kDiagThreads + t + 128];
  __syncthreads();
  if (t < 64) {
    float v[RM];
#pragma unroll
    for (int q = 0; q < RM; ++q) v[q] = red[q * kDiagThreads + t] + red[q * kDiagThreads + t + 64];
#pragma unroll
    for (int h = 32; h > 0; h >>= 1)
#pragma unroll
      for (int q = 0; q < RM; ++q) v[q] += __shfl_down(v[q], h, 64);
    if (t == 0)
#pragma unroll
      for (int q = 0; q < RM; ++q)
        if (q < g.r) g.out[((int64_t)s * g.Nt + i) * g.r + q] = v[q];
  }
}
// C == 1: block (tile of 64 consecutive i, slice of a); lane <-> i (contiguous in Y), the
// four waves stride over a and their sums are added in wave order.  A wave issues the loads
// of kU steps of a before their products (each accumulator still takes its terms in
// ascending a); the rank index of a load is clamped instead of guarded, so no load waits on
// a branch (accumulators past r are never stored), and lanes past Nt read row Nt - 1 and
// are not stored either.
template <int RM, bool GRAM>
__global__ __launch_bounds__(kDiagThreads) void diag_outer_k(DiagArgs g) {
  __shared__ float red[kDiagThreads * RM];
  if constexpr (GRAM)
    if (diag_gram<RM>(g, red)) return;
  const int block = blockIdx.x - (GRAM ? 1 : 0);
  const int64_t tiles = (g.Nt + 63) / 64;
  const int64_t tile = block % tiles;
  const int s = (int)(block / tiles);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = tile * 64 + lane;
  const int64_t ic = i < g.Nt ? i : g.Nt - 1;
  const int64_t a0 = g.A * s / g.slices, a1 = g.A * (s + 1) / g.slices;
  constexpr int kW = kDiagThreads / 64;
  constexpr int kU = RM <= 16 ? 4 : 2;
  // rank entry q of row a for this lane: Y[(a Nt + i) r + q] (rank last) or
  // Y[q A Nt + a Nt + i] (rank first)
  const int64_t qstride = g.rho_first ? g.A * g.Nt : 1;
  const int64_t astride = g.rho_first ? g.Nt : g.Nt * g.r;
  const float *ylane = g.Y + (g.rho_first ? ic : ic * g.r);
  float acc[RM];
#pragma unroll
  for (int q = 0; q < RM; ++q) acc[q] = 0.f;
  for (int64_t ab = a0 + w; ab < a1; ab += kU * kW) {
    float y[kU][RM], wt[kU][RM];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t a = ab + u * kW;
      const int64_t ac = a < a1 ? a : a1 - 1;
      const float *yr = ylane + ac * astride;
#pragma unroll
      for (int q = 0; q < RM; ++q) {
        const int qc = q < g.r ? q : g.r - 1;
        y[u][q] = yr[qc * qstride];
        wt[u][q] = diag_w(g, ac, 0, qc);
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const bool ok = ab + u * kW < a1;
#pragma unroll
      for (int q = 0; q < RM; ++q) {
        const float t = fmaf(y[u][q], wt[u][q], acc[q]);
        acc[q] = ok ? t : acc[q];
      }
    }
  }
#pragma unroll
  for (int q = 0; q < RM; ++q) red[(w * RM + q) * 64 + lane] = acc[q];
  __syncthreads();
  for (int idx = threadIdx.x; idx < RM * 64; idx += kDiagThreads) {
    const int q = idx >> 6, l = idx & 63;
    const int64_t ii = tile * 64 + l;
    if (q >= g.r || ii >= g.Nt) continue;
    float t = red[q * 64 + l];
    for (int ww = 1; ww < kW; ++ww) t += red[(ww * RM + q) * 64 + l];
    g.out[((int64_t)s * g.Nt + ii) * g.r + q] = t;
  }
}
int64_t diag_slices(int64_t A, int64_t Nt, int64_t C) {
  if (C > 1) {
    const int64_t per = std::max<int64_t>(1, 512 / Nt);
    return std::max<int64_t>(1, std::min<int64_t>(per, (A * C) / (kDiagThreads * 4)));
  }
  const int64_t tiles = (Nt + 63) / 64;
  const int64_t per = std::max<int64_t>(1, 512 / tiles);
  return std::max<int64_t>(1, std::min<int64_t>(per, A / 16));
}

// A Gram by the diagonal contraction's extra block takes about as long as the contraction up to here
// (512 rows at rank 10: hidden; gram_block_k 5.1 us); below rank 4 most of its tiles would be padding.
bool diag_gram_fits(int64_t N, int r) { return N <= 1024 && r >= 4; }

nnc_status launch_diag(const float *Y, int rho_first, int64_t A, int64_t Nt, int64_t C, const float *WA,
                       const float *WC, int r, float *part, const float *gB, int64_t gN, float *gS, hipStream_t s) {
  if (r < 1 || r > 32) return fail(NNC_EUNSUPPORTED, "rank %d outside [1, 32]", r);
  const int64_t S = diag_slices(A, Nt, C);
  if (!part) return fail(NNC_EINVAL, "diag: partial buffer missing");
  if (gB && !diag_gram_fits(gN, r)) return fail(NNC_EUNSUPPORTED, "diag: Gram of %lld rows at rank %d", (long long)gN, r);
  DiagArgs g{Y, WA, WC, A, Nt, C, r, rho_first, part, (int)S, gB, gS, (int)gN};
  const int64_t blocks = (C > 1 ? Nt * S : ((Nt + 63) / 64) * S) + (gB ? 1 : 0);
  if (blocks > 0x7fffffff) return fail(NNC_EUNSUPPORTED, "diag: grid too large");
  const int RM = r <= 8 ? 8 : (r <= 16 ? 16 : 32);
#define NNC_DIAG2(KERN, GRAM)                                                                                        \
  do {                                                                                                               \
    if (RM == 8) hipLaunchKernelGGL((KERN<8, GRAM>), dim3((unsigned)blocks), dim3(kDiagThreads), 0, s, g);           \
    else if (RM == 16) hipLaunchKernelGGL((KERN<16, GRAM>), dim3((unsigned)blocks), dim3(kDiagThreads), 0, s, g);    \
    else hipLaunchKernelGGL((KERN<32, GRAM>), dim3((unsigned)blocks), dim3(kDiagThreads), 0, s, g);                  \
  } while (0)
#define NNC_DIAG(KERN)        \
  do {                        \
    if (gB)                   \
      NNC_DIAG2(KERN, true);  \
    else                      \
      NNC_DIAG2(KERN, false); \
  } while (0)
  if (C > 1) NNC_DIAG(diag_inner_k);
  else NNC_DIAG(diag_outer_k);
#undef NNC_DIAG2
#undef NNC_DIAG
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

int64_t diag_part_floats(int64_t A, int64_t Nt, int64_t C, int r) {
  const int64_t S = diag_slices(A, Nt, C);
  return S * Nt * r;
}

// B <- B * M / max(B H, eps) with M = sum_{s < slices} part[s] (s in order) and H = prod_{k != n} S_k
// (entrywise, S packed [d][r][r]); FP64 division, clipped denominators counted.  Thread (row, rho),
// 256 / r rows per block.  Bound by the latency of one round of loads: 4.8 us at 512 x 10 and 64 slices
// (the sum and the update as two launches: 10.0).  kB slices are read together: as many as a few rounds
// take, and one where there is only one (20 x 3: 0.8 us less than with 32 reads of it).
template <int kB>
__global__ __launch_bounds__(256) void cp_mu_k(float *__restrict__ B, const float *__restrict__ part, int slices,
                                               const float *__restrict__ S, int d, int n, int64_t N,
                                               int r, double eps, unsigned long long *clips) {
  __shared__ float H[32 * 32];
  __shared__ unsigned int nclip;
  const int tid = threadIdx.x;
  const int rpb = 256 / r;
  const int64_t i = (int64_t)blockIdx.x * rpb + tid / r;
  const int q = tid % r;
  const bool act = tid < rpb * r && i < N;
  // the loads of a group of slices are all in flight before the adds, the first group's (and the row's)
  // beside those of H; a slice past the last is read as the last and added as zero
  constexpr int kR = 8;
  const int64_t n1 = N * r;
  const float *pe = part + (act ? i * r + q : 0);
  float v[kB], row[kR];
#pragma unroll
  for (int k = 0; k < kB; ++k) v[k] = pe[(int64_t)min(k, slices - 1) * n1];
  const float *br = B + (act ? i * r : 0);
#pragma unroll
  for (int t = 0; t < kR; ++t) row[t] = br[min(t, r - 1)];
  const float old = br[act ? q : 0];
  for (int e = tid; e < r * r; e += 256) {
    float h = 1.f;
    for (int k = 0; k < d; ++k)
      if (k != n) h *= S[(int64_t)k * r * r + e];
    H[e] = h;
  }
  if (tid == 0) nclip = 0;
  float m = v[0];
#pragma unroll
  for (int k = 1; k < kB; ++k) m += k < slices ? v[k] : 0.f;
  for (int s = kB; s < slices; s += kB) {
#pragma unroll
    for (int k = 0; k < kB; ++k) v[k] = pe[(int64_t)min(s + k, slices - 1) * n1];
#pragma unroll
    for (int k = 0; k < kB; ++k) m += s + k < slices ? v[k] : 0.f;
  }
  __syncthreads();
  float nv = 0.f;
  unsigned int mine = 0;
  if (act) {
    float den = 0.f;
#pragma unroll
    for (int t = 0; t < kR; ++t)
      if (t < r) den = fmaf(row[t], H[t * r + q], den);
    for (int t = kR; t < r; ++t) den = fmaf(br[t], H[t * r + q], den);
    double dd = (double)den;
    if (dd < eps) {
      dd = eps;
      mine = 1;
    }
    nv = (float)(((double)old * (double)m) / dd);
  }
  if (mine) atomicAdd(&nclip, mine);
  __syncthreads();  // every row of the block is read before any is written
  if (act) B[i * r + q] = nv;
  if (tid == 0 && nclip) atomicAdd(clips, (unsigned long long)nclip);
}

nnc_status launch_cp_mu(float *B, const float *part, int64_t slices, const float *S, int d, int n, int64_t N, int r,
                        double eps, unsigned long long *clips, hipStream_t s) {
  if (r < 1 || r > 32) return fail(NNC_EUNSUPPORTED, "rank %d outside [1, 32]", r);
  const int64_t rpb = 256 / r;
#define NNC_CP_MU(KB)                                                                                            \
  hipLaunchKernelGGL(cp_mu_k<KB>, dim3((unsigned)((N + rpb - 1) / rpb)), dim3(256), 0, s, B, part, (int)slices, S, d, n, \
                     N, r, eps, clips)
  if (slices == 1)
    NNC_CP_MU(1);
  else if (slices <= 8)
    NNC_CP_MU(8);
  else
    NNC_CP_MU(32);
#undef NNC_CP_MU
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

// S = A^T A (A: N x r, r <= 32) in one workgroup: thread (entry, split) sums the rows of its
// split (rows j with j mod splits == split) in ascending order, the splits are added in
// order.  Rows come through LDS in chunks of a multiple of `splits` rows, each chunk one
// round of coalesced loads: read from global memory, the sum waited on one load latency per
// few rows.
constexpr int kGramLds = 8192;  // floats of A staged per chunk
static __device__ void gram_block_body(const float *__restrict__ A, int64_t N, int r, float *__restrict__ S) {
  __shared__ float part[1024];
  __shared__ float As[kGramLds];
  const int tid = threadIdx.x;
  const int rr = r * r;
  const int splits = 1024 / rr;
  const int e = tid % rr, sp = tid / rr;
  const int a = e / r, b = e - (e / r) * r;
  const int64_t crows = (int64_t)(kGramLds / r / splits) * splits;  // rows per chunk
  float acc = 0.f;
  for (int64_t c0 = 0; c0 < N; c0 += crows) {
    const int64_t nrow = N - c0 < crows ? N - c0 : crows;
    const int nv = (int)(nrow * r);
    __syncthreads();  // the previous chunk is consumed
    constexpr int kPer = kGramLds / 1024;
    float v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = tid + u * 1024;
      v[u] = A[c0 * r + (i < nv ? i : 0)];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = tid + u * 1024;
      if (i < nv) As[i] = v[u];
    }
    __syncthreads();
    if (sp < splits) {
#pragma unroll 8
      for (int j = sp; j < nrow; j += splits) acc = fmaf(As[j * r + a], As[j * r + b], acc);
    }
  }
  part[tid] = acc;
  __syncthreads();
  if (tid < rr) {
    float t = part[tid];
    for (int k = 1; k < splits; ++k) t += part[k * rr + tid];
    S[tid] = t;
  }
}

__global__ __launch_bounds__(1024) void gram_block_k(const float *__restrict__ A, int64_t N, int r,
                                                     float *__restrict__ S) {
  gram_block_body(A, N, r, S);
}

// The Grams of several factors at once, block k taking factor k.
struct GramSet {
  const float *A[kMaxDim];
  float *S[kMaxDim];
  int64_t N[kMaxDim];
  int r[kMaxDim];
};
__global__ __launch_bounds__(1024) void gram_set_k(GramSet g) {
  const int k = blockIdx.x;
  const float *A = nullptr;
  float *S = nullptr;
  int64_t N = 0;
  int r = 1;
#pragma unroll
  for (int j = 0; j < kMaxDim; ++j)  // selects by unrolled compares: no dynamic argument indexing
    if (j == k) {
      A = g.A[j];
      S = g.S[j];
      N = g.N[j];
      r = g.r[j];
    }
  gram_block_body(A, N, r, S);
}

nnc_status launch_gram_block(const float *A, int64_t N, int r, float *S, hipStream_t s) {
  if (r < 1 || r > 32) return fail(NNC_EUNSUPPORTED, "rank %d outside [1, 32]", r);
  hipLaunchKernelGGL(gram_block_k, dim3(1), dim3(1024), 0, s, A, N, r, S);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

nnc_status launch_gram_set(int d, const float *const *A, const int64_t *N, const int64_t *R, float *const *S,
                           hipStream_t s) {
  GramSet g;
  memset(&g, 0, sizeof g);
  for (int k = 0; k < d; ++k) {
    if (R[k] < 1 || R[k] > 32) return NNC_EUNSUPPORTED;
    g.A[k] = A[k];
    g.S[k] = S[k];
    g.N[k] = N[k];
    g.r[k] = (int)R[k];
  }
  hipLaunchKernelGGL(gram_set_k, dim3(d), dim3(1024), 0, s, g);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

// out[j][i] = in[i][j] (rows x cols -> cols x rows), small matrices.
__global__ void transpose_k(const float *__restrict__ in, int64_t rows, int64_t cols, float *__restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= rows * cols) return;
  const int64_t i = e / cols, j = e - (e / cols) * cols;
  out[j * rows + i] = in[e];
}

nnc_status launch_transpose(const float *in, int64_t rows, int64_t cols, float *out, hipStream_t s) {
  const int64_t n = rows * cols;
  if (n == 0) return NNC_OK;
  hipLaunchKernelGGL(transpose_k, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, in, rows, cols, out);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc

namespace nnc {

// =====================================================================================
// NMF A ~ W H (Lee-Seung multiplicative sweeps, W first, then H) of up to kNmfMax
// independent problems with a common column count, one workgroup per problem with A, W, H
// and the small products in LDS:
//   G = H H^T;  W <- W * (A H^T) / max(W G, eps)          (a thread per row of W)
//   G = W^T W, P = W^T A                                    (a thread per (column j of W,
//                                                            row range), ranges added in order)
//   H <- H * P / max(G H, eps).
// A is rows x cols, W rows x m, H m x cols; FP32 products, FP64 divisions, clipped
// denominators counted; ||A - W H||^2 and ||A||^2 in FP64 at the end.  RC / MC bound cols / m
// (8, 16 or 32) so that a row of A, of W and its new values stay in registers.
// =====================================================================================
constexpr int kNmfMax = 8;
constexpr int kNmfThreads = 512;
constexpr int kNmfSplitMax = 32;
constexpr size_t kNmfLdsMax = 159 * 1024;  // dynamic LDS; the static part (counters) stays below 1 KiB

struct NmfArgs {
  const float *A[kNmfMax];
  float *W[kNmfMax];
  float *H[kNmfMax];
  int rows[kNmfMax], m[kNmfMax];
  int cols, iters;
  double eps;
  unsigned long long *clips;
  double *red;  // [problem][2] (||A - W H||^2, ||A||^2) or null
};

__host__ __device__ static inline int nmf_splits(int m) { return kNmfThreads / m < kNmfSplitMax ? kNmfThreads / m : kNmfSplitMax; }

static inline int pad4(int x) { return (x + 3) & ~3; }

// LDS floats: A [rows][rp] | W [rows][mp] | H [m][rp] | P [m][rp] | G [m][mp] |
// partial sums [splits][m][mp + rp]   (rp, mp: cols and m rounded up to 4, zero padding)
size_t nmf_lds_floats(int rows, int cols, int m) {
  const size_t rp = pad4(cols), mp = pad4(m);
  return (size_t)rows * (rp + mp) + 2 * (size_t)m * rp + (size_t)m * mp + (size_t)nmf_splits(m) * m * (mp + rp);
}

bool nmf_block_fits(int rows, int cols, int m) {
  return cols <= 32 && m <= 32 && nmf_lds_floats(rows, cols, m) * 4 <= kNmfLdsMax;
}

static __device__ inline float dot4(float4 a, float4 b, float s) {
  s = fmaf(a.x, b.x, s);
  s = fmaf(a.y, b.y, s);
  s = fmaf(a.z, b.z, s);
  return fmaf(a.w, b.w, s);
}

// red[2 b], red[2 b + 1] <- ||A - W H||^2, ||A||^2 in FP64 of the workgroup's problem, if asked for
// (a barrier inside; every thread takes part)
static __device__ inline void nmf_residual(const float *A, int as, const float *W, int ws, const float *H, int hs, int N, int r, int m,
                                           int b, double *red, double (*dred)[kNmfThreads / 64]) {
  if (!red) return;
  const int tid = threadIdx.x;
  double se = 0.0, sa = 0.0;
  for (int e = tid; e < N * r; e += kNmfThreads) {
    const int i = e / r, q = e - (e / r) * r;
    float x = 0.f;
    for (int k = 0; k < m; ++k) x = fmaf(W[i * ws + k], H[k * hs + q], x);
    const float av = A[i * as + q];
    const double dlt = (double)av - (double)x;
    se += dlt * dlt;
    sa += (double)av * (double)av;
  }
  for (int off = 32; off > 0; off >>= 1) {
    se += __shfl_down(se, off);
    sa += __shfl_down(sa, off);
  }
  if ((tid & 63) == 0) {
    dred[0][tid >> 6] = se;
    dred[1][tid >> 6] = sa;
  }
  __syncthreads();
  if (tid == 0) {
    double a = 0.0, c = 0.0;
    for (int w = 0; w < kNmfThreads / 64; ++w) {
      a += dred[0][w];
      c += dred[1][w];
    }
    red[2 * b] = a;
    red[2 * b + 1] = c;
  }
}

template <int RC, int MC>
__global__ __launch_bounds__(kNmfThreads) void nmf_block_k(NmfArgs g) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ unsigned int nclip;
  __shared__ double dred[2][kNmfThreads / 64];
  constexpr int R4 = RC / 4, M4 = MC / 4;
  const int b = blockIdx.x, tid = threadIdx.x;
  const int N = g.rows[b], m = g.m[b], r = g.cols;
  const int rp = (r + 3) & ~3, mp = (m + 3) & ~3, rq = rp / 4, mq = mp / 4;
  const float *__restrict__ Ag = g.A[b];
  float *__restrict__ Wg = g.W[b];
  float *__restrict__ Hg = g.H[b];
  const int S = nmf_splits(m), O = mp + rp;
  float *A = sm, *W = A + N * rp, *H = W + N * mp, *P = H + m * rp, *G = P + m * rp, *part = G + m * mp;
  for (int e = tid; e < N * rp; e += kNmfThreads) {
    const int i = e / rp, q = e - (e / rp) * rp;
    A[e] = q < r ? Ag[i * r + q] : 0.f;
  }
  for (int e = tid; e < N * mp; e += kNmfThreads) {
    const int i = e / mp, k = e - (e / mp) * mp;
    W[e] = k < m ? Wg[i * m + k] : 0.f;
  }
  for (int e = tid; e < m * rp; e += kNmfThreads) {
    const int j = e / rp, q = e - (e / rp) * rp;
    H[e] = q < r ? Hg[j * r + q] : 0.f;
    P[e] = 0.f;
  }
  for (int e = tid; e < m * mp; e += kNmfThreads) G[e] = 0.f;  // the padding stays zero
  if (tid == 0) nclip = 0;
  __syncthreads();
  unsigned int mine = 0;
  const double eps = g.eps;
  auto mu = [&](float x, float num, float den) {
    double dd = (double)den;
    if (dd < eps) {
      dd = eps;
      ++mine;
    }
    return (float)(((double)x * (double)num) / dd);
  };
  const float4 *A4 = reinterpret_cast<const float4 *>(A);
  const float4 *H4 = reinterpret_cast<const float4 *>(H);
  const float4 *G4 = reinterpret_cast<const float4 *>(G);
  const float4 *W4 = reinterpret_cast<const float4 *>(W);
  const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int it = 0; it < g.iters; ++it) {
    // Rows are read four entries at a time.  Loops run to the compile-time bounds RC / MC
    // with the group index clamped; a group past the row is multiplied by zeros (the
    // padded registers) or replaced by zeros, never guarded by a branch.
    for (int e = tid; e < m * m; e += kNmfThreads) {  // G = H H^T (symmetric)
      const int j = e / m, k = e - (e / m) * m;
      float sacc = 0.f;
#pragma unroll
      for (int q4 = 0; q4 < R4; ++q4) {
        const int qq = q4 < rq ? q4 : rq - 1;
        const float4 hj = H4[j * rq + qq];
        sacc = dot4(q4 < rq ? hj : z4, H4[k * rq + qq], sacc);
      }
      G[j * mp + k] = sacc;
    }
    __syncthreads();
#pragma unroll 1
    for (int i = tid; i < N; i += kNmfThreads) {  // row i of W
      float4 a[R4], w[M4];
#pragma unroll
      for (int q4 = 0; q4 < R4; ++q4) {
        const float4 v = A4[i * rq + (q4 < rq ? q4 : rq - 1)];
        a[q4] = q4 < rq ? v : z4;
      }
#pragma unroll
      for (int k4 = 0; k4 < M4; ++k4) {
        const float4 v = W4[i * mq + (k4 < mq ? k4 : mq - 1)];
        w[k4] = k4 < mq ? v : z4;
      }
#pragma unroll 1
      for (int j = 0; j < m; ++j) {
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int q4 = 0; q4 < R4; ++q4) num = dot4(a[q4], H4[j * rq + (q4 < rq ? q4 : rq - 1)], num);
#pragma unroll
        for (int k4 = 0; k4 < M4; ++k4)  // G[k][j] = G[j][k]
          den = dot4(w[k4], G4[j * mq + (k4 < mq ? k4 : mq - 1)], den);
        // the row belongs to this thread alone: entry j still holds its old value
        W[i * mp + j] = mu(W[i * mp + j], num, den);
      }
    }
    __syncthreads();
    if (tid < S * m) {  // column j of W against rows [i0, i1) of W and A
      const int j = tid % m, sp = tid / m;
      const int i0 = N * sp / S, i1 = N * (sp + 1) / S;
      float4 acc[M4 + R4];
#pragma unroll
      for (int o = 0; o < M4 + R4; ++o) acc[o] = z4;
#pragma unroll 1
      for (int i = i0; i < i1; ++i) {  // accumulators past the row collect unused values
        const float wj = W[i * mp + j];
#pragma unroll
        for (int k4 = 0; k4 < M4; ++k4) {
          const float4 v = W4[i * mq + (k4 < mq ? k4 : mq - 1)];
          acc[k4].x = fmaf(wj, v.x, acc[k4].x);
          acc[k4].y = fmaf(wj, v.y, acc[k4].y);
          acc[k4].z = fmaf(wj, v.z, acc[k4].z);
          acc[k4].w = fmaf(wj, v.w, acc[k4].w);
        }
#pragma unroll
        for (int q4 = 0; q4 < R4; ++q4) {
          const float4 v = A4[i * rq + (q4 < rq ? q4 : rq - 1)];
          acc[M4 + q4].x = fmaf(wj, v.x, acc[M4 + q4].x);
          acc[M4 + q4].y = fmaf(wj, v.y, acc[M4 + q4].y);
          acc[M4 + q4].z = fmaf(wj, v.z, acc[M4 + q4].z);
          acc[M4 + q4].w = fmaf(wj, v.w, acc[M4 + q4].w);
        }
      }
      float4 *pp = reinterpret_cast<float4 *>(part + (sp * m + j) * O);
#pragma unroll
      for (int k4 = 0; k4 < M4; ++k4)
        if (k4 < mq) pp[k4] = acc[k4];
#pragma unroll
      for (int q4 = 0; q4 < R4; ++q4)
        if (q4 < rq) pp[mq + q4] = acc[M4 + q4];
    }
    __syncthreads();
    for (int e = tid; e < m * (m + r); e += kNmfThreads) {  // splits added in order
      const int j = e / (m + r), o = e - (e / (m + r)) * (m + r);
      const int col = o < m ? o : mp + (o - m);
      float t = part[j * O + col];
#pragma unroll
      for (int sp = 1; sp < kNmfSplitMax; ++sp) {  // adding 0 past S changes nothing
        const float v = part[((sp < S ? sp : S - 1) * m + j) * O + col];
        t += sp < S ? v : 0.f;
      }
      if (o < m) G[j * mp + o] = t;
      else P[j * rp + (o - m)] = t;
    }
    __syncthreads();
    // H <- H * (W^T A) / max(W^T W H, eps): m * cols <= 1024 entries, kHv per thread
    constexpr int kHv = (32 * 32 + kNmfThreads - 1) / kNmfThreads;
    float hv[kHv];
#pragma unroll
    for (int u = 0; u < kHv; ++u) {
      const int e = tid + u * kNmfThreads;
      hv[u] = 0.f;
      if (e < m * r) {
        const int j = e / r, q = e - (e / r) * r;
        float den = 0.f;
#pragma unroll
        for (int k = 0; k < MC; ++k) {
          const int kk = k < m ? k : m - 1;
          den = fmaf(k < m ? G[j * mp + kk] : 0.f, H[kk * rp + q], den);
        }
        hv[u] = mu(H[j * rp + q], P[j * rp + q], den);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kHv; ++u) {
      const int e = tid + u * kNmfThreads;
      if (e < m * r) H[(e / r) * rp + e % r] = hv[u];
    }
    __syncthreads();
  }
  for (int e = tid; e < N * m; e += kNmfThreads) Wg[e] = W[(e / m) * mp + e % m];
  for (int e = tid; e < m * r; e += kNmfThreads) Hg[e] = H[(e / r) * rp + e % r];
  if (mine) atomicAdd(&nclip, mine);
  nmf_residual(A, rp, W, mp, H, rp, N, r, m, b, g.red, dred);
  __syncthreads();
  if (tid == 0 && nclip) atomicAdd(g.clips, (unsigned long long)nclip);
}

// =====================================================================================
// The same sweeps on the FP32 matrix cores, for problems whose padded layout fits the LDS: rows to
// a multiple of 16, ranks to 4 MS and columns to 4 QS (zeros), strides an odd number of quads (16
// rows' reads from 64 different banks), all known when compiled.  A sweep is five phases:
//   G = H H^T                                                   (one 16 x 16 tile a wave)
//   W <- W * (A H^T) / max(W G, eps)                            (16 rows of W a wave at a time)
//   [W^T W | W^T A] over row ranges                             (NB ranges a wave at a time)
//   the ranges' sums added in order: G2 to LDS, P to the thread of H's entry
//   H <- H * P / max(G2 H, eps), into H's other buffer.
// Each entry of a product is one accumulator's chain in the order of the contracted index, and a
// 16 x 16 x 4 step adds its four products one after the other: the sums are those of nmf_block_k,
// bit for bit (the iteration is not contracting: another order moves the result of a few hundred
// sweeps by more than rounding).  One quad of ranks past a multiple of 16 (m = 17 .. 20) has its
// part of the W step on the VALU, a value a lane, instead of a second tile of three quarters zeros.
// Bound: instruction issue and latency in one CU: three 512 x 10 at m = 20, 8.4 us a sweep in this
// form, 26.2 in nmf_block_k.
// =====================================================================================
constexpr int kNmfWaves = kNmfThreads / 64;

template <int MS, int QS>
struct NmfMM {
  static constexpr int odd4(int q) { return 4 * (q | 1); }
  static constexpr int M = 4 * MS, Q = 4 * QS, ms = odd4(MS), rs = odd4(QS), os = odd4(MS + QS);
  static constexpr int H = M * rs;            // one of H's two buffers
  static constexpr int dump = 4 * ms + 64;    // values of padded ranks go here
  static size_t floats(int rows, int m) {
    const size_t n16 = (rows + 15) & ~15;
    return n16 * (rs + ms) + 2 * H + M * ms + dump + (size_t)nmf_splits(m) * m * os;
  }
};

template <int MS, int QS>
__global__ __launch_bounds__(kNmfThreads) void nmf_mm_k(NmfArgs g) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ unsigned int nclip;
  __shared__ int range[kNmfSplitMax + 1];
  __shared__ double dred[2][kNmfWaves];
  typedef float f4 __attribute__((ext_vector_type(4)));
  using L = NmfMM<MS, QS>;
  constexpr bool kTail = MS % 4 == 1;
  constexpr int MW = kTail ? MS / 4 : (MS + 3) / 4;  // 16-wide tiles: ranks in the W step, ranks, ranks and columns
  constexpr int MT = (MS + 3) / 4, CT = (MS + QS + 3) / 4;
  constexpr int ms = L::ms, rs = L::rs, os = L::os;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = g.rows[b], m = g.m[b], r = g.cols, S = nmf_splits(m), n16 = (N + 15) & ~15;
  const float *__restrict__ Ag = g.A[b];
  float *__restrict__ Wg = g.W[b];
  float *__restrict__ Hg = g.H[b];
  float *A = sm, *W = A + n16 * rs, *H0 = W + n16 * ms, *G = H0 + 2 * L::H, *dump = G + L::M * ms, *part = dump + L::dump;
  auto mfma = [](float x, float y, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); };
  const f4 zero = f4{0.f, 0.f, 0.f, 0.f};
  for (int e = tid; e < n16 * rs; e += kNmfThreads) {
    const int i = e / rs, q = e - i * rs;
    A[e] = i < N && q < r ? Ag[i * r + q] : 0.f;
  }
  for (int e = tid; e < n16 * ms; e += kNmfThreads) {
    const int i = e / ms, k = e - i * ms;
    W[e] = i < N && k < m ? Wg[i * m + k] : 0.f;
  }
  for (int e = tid; e < L::H; e += kNmfThreads) {
    const int j = e / rs, q = e - j * rs;
    H0[e] = j < m && q < r ? Hg[j * r + q] : 0.f;
    H0[L::H + e] = 0.f;
  }
  for (int e = tid; e < L::M * ms; e += kNmfThreads) G[e] = 0.f;
  if (tid <= S) range[tid] = N * tid / S;
  if (tid == 0) nclip = 0;
  __syncthreads();
  unsigned int mine = 0;
  const double eps = g.eps;
  float eps_up = (float)eps;  // den < eps in double if and only if den < eps_up: the float at or above it
  if ((double)eps_up < eps) eps_up = nextafterf(eps_up, INFINITY);
  const unsigned int lowest = __float_as_uint(fmaxf(eps_up, 1e-37f));  // and normal
  const bool clip_all = eps_up > 3.4028234e38f;                        // no float is as large
  auto mu = [&](float x, float num, float den, bool valid) {
    const bool low = den < eps_up;
    mine += low && valid;
    return (float)(((double)x * (double)num) / (low ? eps : (double)den));
  };
  // the thread's entries of the sums: P's (tid + 512 u < m r), then the upper triangle of G
  constexpr int kHv = (L::M * L::Q + kNmfThreads - 1) / kNmfThreads;
  constexpr int kSv = (L::M * L::Q + L::M * (L::M + 1) / 2 + kNmfThreads - 1) / kNmfThreads;
  const int mr = m * r;
  int sum_at[kSv], sum_j[kSv], sum_c[kSv];  // its place, row and column
#pragma unroll
  for (int u = 0; u < kSv; ++u) {
    const int e = tid + u * kNmfThreads;
    sum_at[u] = -1;
    sum_j[u] = sum_c[u] = 0;
    if (e < mr) {
      sum_j[u] = e / r;
      sum_c[u] = e - sum_j[u] * r;
      sum_at[u] = sum_j[u] * os + L::M + sum_c[u];
    } else if (e < mr + m * (m + 1) / 2) {
      int t = e - mr, j = 0;
      while (t >= m - j) t -= m - j++;
      sum_j[u] = j;
      sum_c[u] = j + t;
      sum_at[u] = j * os + j + t;
    }
  }
  const float *col[CT];  // the lane's columns of [W | A]
  int by[CT];            // and how far apart their rows are
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int o = 16 * c + li;
    col[c] = (o < L::M ? W + o : A + min(o - L::M, rs - 1)) + lg * (o < L::M ? ms : rs);
    by[c] = o < L::M ? ms : rs;
  }
  for (int it = 0; it < g.iters; ++it) {
    const float *H = H0 + (it & 1) * L::H;
    float *Hn = H0 + ((it & 1) ^ 1) * L::H;
    // ---- G = H H^T (H's rows past 4 MS: other parts of the LDS, for rows and columns that are not stored)
    if (wave < MT * MT) {
      const int ma = wave / MT, mb = wave % MT;
      const float *ha = H + (16 * ma + li) * rs + lg, *hb = H + (16 * mb + li) * rs + lg;
      f4 acc = zero;
#pragma unroll
      for (int s = 0; s < QS; ++s) acc = mfma(ha[4 * s], hb[4 * s], acc);
      if (16 * mb + li < L::M) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (16 * ma + 4 * lg < L::M) G[(16 * ma + 4 * lg + k) * ms + 16 * mb + li] = acc[k];
      }
    }
    __syncthreads();
    // ---- W
    {
      f4 th[kTail ? QS : 1], tg[kTail ? MS : 1];
      const int tj = 16 * MW + (lane & 3);  // the lane's rank of the tail, its row: lane / 4
      float h[QS][MW], gg[MS][MW];
#pragma unroll
      for (int mt = 0; mt < MW; ++mt) {
#pragma unroll
        for (int s = 0; s < QS; ++s) h[s][mt] = H[(16 * mt + li) * rs + 4 * s + lg];
#pragma unroll
        for (int s = 0; s < MS; ++s) gg[s][mt] = G[(16 * mt + li) * ms + 4 * s + lg];  // G is symmetric
      }
      if (kTail) {
#pragma unroll
        for (int s = 0; s < QS; ++s) th[kTail ? s : 0] = *reinterpret_cast<const f4 *>(H + tj * rs + 4 * s);
#pragma unroll
        for (int s = 0; s < MS; ++s) tg[kTail ? s : 0] = *reinterpret_cast<const f4 *>(G + tj * ms + 4 * s);
      }
      for (int t = wave; 16 * t < N; t += kNmfWaves) {
        constexpr int NQ = 4 * MW + (kTail ? 1 : 0);  // the lane's entries of the tile
        const int rd = 16 * t + 4 * lg;
        const float *ap = A + (16 * t + li) * rs + lg, *wp = W + (16 * t + li) * ms + lg;
        float *xp = W + rd * ms + li;
        float a[QS], w[MS], q_x[NQ], q_num[NQ], q_den[NQ];
        bool q_in[NQ];
#pragma unroll
        for (int s = 0; s < QS; ++s) a[s] = ap[4 * s];
#pragma unroll
        for (int s = 0; s < MS; ++s) w[s] = wp[4 * s];
#pragma unroll
        for (int u = 0; u < 4 * MW; ++u) q_x[u] = xp[(u & 3) * ms + 16 * (u >> 2)];
        f4 num[MW], den[MW];
#pragma unroll
        for (int mt = 0; mt < MW; ++mt) num[mt] = den[mt] = zero;
#pragma unroll
        for (int s = 0; s < (MS > QS ? MS : QS); ++s) {
          if (s < QS) {
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) num[mt] = mfma(a[s < QS ? s : 0], h[s < QS ? s : 0][mt], num[mt]);
          }
          if (s < MS) {
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) den[mt] = mfma(w[s < MS ? s : 0], gg[s < MS ? s : 0][mt], den[mt]);
          }
        }
        if (kTail) {
          const int row = 16 * t + (lane >> 2);
          float tn = 0.f, td = 0.f;
#pragma unroll
          for (int s = 0; s < QS; ++s) {
            const f4 v = *reinterpret_cast<const f4 *>(A + row * rs + 4 * s);
#pragma unroll
            for (int u = 0; u < 4; ++u) tn = fmaf(v[u], th[kTail ? s : 0][u], tn);
          }
#pragma unroll
          for (int s = 0; s < MS; ++s) {
            const f4 v = *reinterpret_cast<const f4 *>(W + row * ms + 4 * s);
#pragma unroll
            for (int u = 0; u < 4; ++u) td = fmaf(v[u], tg[kTail ? s : 0][u], td);
          }
          q_x[NQ - 1] = W[row * ms + tj];
          q_num[NQ - 1] = tn;
          q_den[NQ - 1] = td;
          q_in[NQ - 1] = tj < m && row < N;
        }
#pragma unroll
        for (int u = 0; u < 4 * MW; ++u) {
          q_num[u] = num[u >> 2][u & 3];
          q_den[u] = den[u >> 2][u & 3];
          q_in[u] = 16 * (u >> 2) + li < m && rd + (u & 3) < N;
        }
        // All quotients of the lane at once, a step of every chain after the other (one by one they are a
        // serial chain of a dozen FP64 operations each).  The reciprocal is the hardware's estimate and two
        // Newton steps, within an ulp or two of double precision, and the quotient is corrected by its
        // remainder, which makes the float that of a division: the numerator is a product of two floats and
        // the denominator a float, so a quotient that is not a rounding boundary of the floats (25 bits)
        // itself lies at least 2^-49 of its size from it, and one that is comes out exact.  Denominators to
        // clip, subnormal, infinite or NaN, and numerators that are infinite or NaN, take the division.
        bool odd = clip_all;
        double q_a[NQ];
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
          q_a[u] = (double)q_x[u] * (double)q_num[u];
          odd |= q_in[u] && (__float_as_uint(q_den[u]) - lowest > 0x7f7fffffu - lowest || !__builtin_isfinite(q_a[u]));
        }
        float v[NQ];
        if (__any(odd)) {
#pragma unroll
          for (int u = 0; u < NQ; ++u) v[u] = mu(q_x[u], q_num[u], q_den[u], q_in[u]);
        } else {
          double q[NQ], t[NQ];
#pragma unroll
          for (int u = 0; u < NQ; ++u) q[u] = __builtin_amdgcn_rcp((double)q_den[u]);
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < NQ; ++u) q[u] = fma(q[u], fma(-(double)q_den[u], q[u], 1.0), q[u]);
#pragma unroll
          for (int u = 0; u < NQ; ++u) t[u] = q_a[u] * q[u];
#pragma unroll
          for (int u = 0; u < NQ; ++u) v[u] = (float)fma(fma(-(double)q_den[u], t[u], q_a[u]), q[u], t[u]);
        }
        // rows past N may hold anything, ranks past m stay zero
#pragma unroll
        for (int mt = 0; mt < MW; ++mt) {
          float *to = 16 * mt + li < m ? xp + 16 * mt : dump + lane;
#pragma unroll
          for (int k = 0; k < 4; ++k) to[k * ms] = v[4 * mt + k];
        }
        if (kTail) *(tj < m ? W + (16 * t + (lane >> 2)) * ms + tj : dump + lane) = v[NQ - 1];
      }
    }
    __syncthreads();
    // ---- [W^T W | W^T A] of the row ranges, whose lengths differ by at most one
    constexpr int NB = MT * CT <= 4 ? 4 : MT * CT <= 6 ? 2 : 1;
    for (int sp0 = wave; sp0 < S; sp0 += NB * kNmfWaves) {
      f4 acc[NB][MT][CT];
      const float *xp[NB], *yp[NB][CT];
      int left[NB];  // rows of the range from the lane's row of the step
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int sp = min(sp0 + n * kNmfWaves, S - 1), i0 = __builtin_amdgcn_readfirstlane(range[sp]);
        left[n] = __builtin_amdgcn_readfirstlane(range[sp + 1]) - i0 - lg;
        xp[n] = W + (i0 + lg) * ms + li;
#pragma unroll
        for (int c = 0; c < CT; ++c) yp[n][c] = col[c] + i0 * by[c];
      }
      float x[NB][MT], y[NB][CT];
      auto load = [&] {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
#pragma unroll
          for (int p = 0; p < MT; ++p) x[n][p] = xp[n][16 * p];
#pragma unroll
          for (int c = 0; c < CT; ++c) y[n][c] = *yp[n][c];
          xp[n] += 4 * ms;
#pragma unroll
          for (int c = 0; c < CT; ++c) yp[n][c] += 4 * by[c];
        }
      };
      auto step = [&](bool first, bool whole) {  // four rows of each range, the next four on their way
        float u[NB][MT], v[NB][CT];
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const unsigned int in = whole || left[n] > 0 ? 0xffffffffu : 0u;  // rows past the range are others of the LDS
#pragma unroll
          for (int p = 0; p < MT; ++p) u[n][p] = __uint_as_float(__float_as_uint(x[n][p]) & in);
#pragma unroll
          for (int c = 0; c < CT; ++c) v[n][c] = __uint_as_float(__float_as_uint(y[n][c]) & in);
          left[n] -= 4;
        }
        load();
#pragma unroll
        for (int p = 0; p < MT; ++p)
#pragma unroll
          for (int c = p; c < CT; ++c)
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[n][p][c] = mfma(u[n][p], v[n][c], first ? zero : acc[n][p][c]);
      };
      const int whole = N / S & ~3;
      int i = 4;
      load();
      step(true, whole > 0);
      for (; i + 8 <= whole; i += 8) {
        step(false, true);
        step(false, true);
      }
      for (; i < whole; i += 4) step(false, true);
      for (; i < (N + S - 1) / S; i += 4) step(false, false);
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int sp = sp0 + n * kNmfWaves;
        if (sp < S) {
          float *pw = part + sp * m * os + 4 * lg * os + li;
#pragma unroll
          for (int p = 0; p < MT; ++p)
#pragma unroll
            for (int c = p; c < CT; ++c)
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                const bool in = 16 * p + 4 * lg + k < m && 16 * c + li < L::M + L::Q;
                float *to = in ? pw + (16 * p + k) * os + 16 * c : dump + lane;
                *to = acc[n][p][c][k];
              }
        }
      }
    }
    __syncthreads();
    // ---- the ranges' sums in order
    float pv[kHv];
#pragma unroll
    for (int u = 0; u < kSv; ++u)
      if (sum_at[u] >= 0) {
        const float *pp = part + sum_at[u];
        float t = *pp;
#pragma unroll 8
        for (int sp = 1; sp < S; ++sp) t += pp[sp * m * os];
        if (u < kHv && tid + u * kNmfThreads < mr) {
          pv[u < kHv ? u : 0] = t;
        } else {
          G[sum_j[u] * ms + sum_c[u]] = t;
          G[sum_c[u] * ms + sum_j[u]] = t;
        }
      }
    __syncthreads();
    // ---- H
#pragma unroll
    for (int u = 0; u < kHv; ++u)
      if (tid + u * kNmfThreads < mr) {
        const int at = sum_j[u] * rs + sum_c[u];
        float den = 0.f;
#pragma unroll
        for (int k = 0; k < L::M; k += 4) {
          const f4 gk = *reinterpret_cast<const f4 *>(G + sum_j[u] * ms + k);
#pragma unroll
          for (int v = 0; v < 4; ++v) den = fmaf(gk[v], H[(k + v) * rs + sum_c[u]], den);
        }
        Hn[at] = mu(H[at], pv[u], den, true);
      }
    __syncthreads();
  }
  const float *H = H0 + (g.iters & 1) * L::H;
  for (int e = tid; e < N * m; e += kNmfThreads) Wg[e] = W[(e / m) * ms + e % m];
  for (int e = tid; e < m * r; e += kNmfThreads) Hg[e] = H[(e / r) * rs + e % r];
  if (mine) atomicAdd(&nclip, mine);
  nmf_residual(A, rs, W, ms, H, rs, N, r, m, b, g.red, dred);
  __syncthreads();
  if (tid == 0 && nclip) atomicAdd(g.clips, (unsigned long long)nclip);
}

// The forms of nmf_mm_k: ranks up to 16, 20, 24 or 32 by columns up to 8, 12, 16 or 32.
#define NNC_NMF_ALL                                         \
  NNC_NMF(4, 2) NNC_NMF(4, 3) NNC_NMF(4, 4) NNC_NMF(4, 8)   \
  NNC_NMF(5, 2) NNC_NMF(5, 3) NNC_NMF(5, 4) NNC_NMF(5, 8)   \
  NNC_NMF(6, 2) NNC_NMF(6, 3) NNC_NMF(6, 4) NNC_NMF(6, 8)   \
  NNC_NMF(8, 2) NNC_NMF(8, 3) NNC_NMF(8, 4) NNC_NMF(8, 8)

// Raises a kernel's dynamic-LDS limit to kNmfLdsMax, once.
static nnc_status nmf_allow_lds(const void *kernel) {
  static std::mutex mu;
  static std::set<const void *> done;
  std::lock_guard<std::mutex> lk(mu);
  if (done.count(kernel)) return NNC_OK;
  NNC_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kNmfLdsMax));
  done.insert(kernel);
  return NNC_OK;
}

// Few ranks over many rows, where a tile of 16 ranks is mostly padding and its waves' rounds over the
// rows are what a sweep takes: nmf_block_k, a row a thread, gives the same bits sooner (us a sweep here
// and there: 420 x 8 at m = 1 5.0 and 3.6, 512 x 2 at 4 5.5 and 4.6, 300 x 8 at 5 4.2 and 4.1; at up to
// 128 rows, one round, 3.2 and 3.3 or more; 200 x 20 at 4 3.7 and 5.7).
static bool nmf_block_sooner(const NmfArgs &g, int n, int mmax) {
  int rows = 0;
  for (int b = 0; b < n; ++b) rows = std::max(rows, g.rows[b]);
  return (mmax <= 4 && rows > 128 && g.cols <= 16) || (mmax <= 6 && rows > 256 && g.cols <= 8);
}

// Launches the form that holds the largest rank and the columns; false where a problem's padded
// layout does not fit the LDS (many rows), which nmf_block_k with its packed rows then takes, and
// where that is the sooner one.
static bool launch_nmf_mm(const NmfArgs &g, int n, int mmax, hipStream_t s, nnc_status *st) {
  if (nmf_block_sooner(g, n, mmax)) return false;
  const int ms = mmax <= 16 ? 4 : mmax <= 20 ? 5 : mmax <= 24 ? 6 : 8;
  const int qs = g.cols <= 8 ? 2 : g.cols <= 12 ? 3 : g.cols <= 16 ? 4 : 8;
  size_t lds = 0;
#define NNC_NMF(MSV, QSV)        \
  if (ms == MSV && qs == QSV)    \
    for (int b = 0; b < n; ++b) lds = std::max(lds, NmfMM<MSV, QSV>::floats(g.rows[b], g.m[b]) * 4);
  NNC_NMF_ALL
#undef NNC_NMF
  if (lds > kNmfLdsMax) return false;
  auto run = [&](auto *kernel) -> nnc_status {
    NNC_TRY(nmf_allow_lds(reinterpret_cast<const void *>(kernel)));
    hipLaunchKernelGGL(kernel, dim3(n), dim3(kNmfThreads), lds, s, g);
    NNC_HIP(hipGetLastError());
    return NNC_OK;
  };
#define NNC_NMF(MSV, QSV) \
  if (ms == MSV && qs == QSV) *st = run(nmf_mm_k<MSV, QSV>);
  NNC_NMF_ALL
#undef NNC_NMF
  return true;
}

nnc_status launch_nmf_block(int n, const float *const *A, const int *rows, int cols, const int *m,
                            int iters, float *const *W, float *const *H, double eps,
                            unsigned long long *clips, double *red, hipStream_t s) {
  if (n < 1 || n > kNmfMax) return fail(NNC_EUNSUPPORTED, "nmf: %d problems per launch", n);
  NmfArgs g;
  memset(&g, 0, sizeof g);
  size_t lds = 0;
  for (int b = 0; b < n; ++b) {
    if (!nmf_block_fits(rows[b], cols, m[b])) return NNC_EUNSUPPORTED;
    g.A[b] = A[b];
    g.W[b] = W[b];
    g.H[b] = H[b];
    g.rows[b] = rows[b];
    g.m[b] = m[b];
    lds = std::max(lds, nmf_lds_floats(rows[b], cols, m[b]) * 4);
  }
  g.cols = cols;
  g.iters = iters;
  g.eps = eps;
  g.clips = clips;
  g.red = red;
  int mmax = 1;
  for (int k = 0; k < n; ++k) mmax = std::max(mmax, m[k]);
  nnc_status st = NNC_OK;
  if (launch_nmf_mm(g, n, mmax, s, &st)) return st;
  const int RC = cols <= 8 ? 8 : (cols <= 16 ? 16 : 32), MC = mmax <= 8 ? 8 : (mmax <= 16 ? 16 : 32);
#define NNC_NMF(RCV, MCV)                                                                         \
  do {                                                                                            \
    NNC_TRY(nmf_allow_lds(reinterpret_cast<const void *>(nmf_block_k<RCV, MCV>)));                \
    hipLaunchKernelGGL((nmf_block_k<RCV, MCV>), dim3(n), dim3(kNmfThreads), lds, s, g);           \
  } while (0)
#define NNC_NMF_M(RCV)                \
  do {                                \
    if (MC == 8) NNC_NMF(RCV, 8);     \
    else if (MC == 16) NNC_NMF(RCV, 16); \
    else NNC_NMF(RCV, 32);            \
  } while (0)
  if (RC == 8) NNC_NMF_M(8);
  else if (RC == 16) NNC_NMF_M(16);
  else NNC_NMF_M(32);
#undef NNC_NMF_M
#undef NNC_NMF
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc
