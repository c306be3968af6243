// Least-squares steps of the real-valued CANDELINC Tucker fit (Section 2.2: a Tucker
// decomposition of X, then a CPD of its core).  The X passes and the small contractions that
// feed these steps are the nonnegative sweep's kernels; what differs is the update of each
// block, done here in FP64:
//
//   factor n:  A* = num_n K_n^{-1}       (num_n = Y_(n) G_(n)^T, K_n = G_(n) (kron_{k!=n} S_k) G_(n)^T)
//              A* = Q L^T                 (Cholesky QR: L L^T = A*^T A*, Q = A* L^{-T})
//              A_n <- Q,  G <- G x_n L^T, S_n <- Q^T Q
//   core:      G <- (X x_1 A_1^T ... x_d A_d^T) x_1 S_1^{-1} ... x_d S_d^{-1}
//
// The factor step only needs R x R quantities besides two passes over the N x R rows:
//   Z = num^T num,  A*^T A* = K^{-1} Z K^{-1} = L L^T,  T = K^{-1} L^{-T},  Q = num T,
//   Q^T Q = T^T Z T;
// one workgroup forms Z and the R x R algebra (ls_small_k), one launch applies T to the rows and
// L^T to the core (ls_apply_k), and one forms the core step's inverse Grams (ls_inv_k, a block
// each).  R x R inverses come from Gauss-Jordan elimination without pivoting: its pivots are those
// of the LDL^T factorization, positive exactly when the matrix is positive definite, so a pivot
// that is not positive marks a system that is not (counted in `fails`).  Every sum runs in a fixed
// order, so results are reproducible.
//
// ls_small_k is a chain of R x R steps that no other work hides, so its length is what counts: the
// inverse of K (one wave, a row a lane, no barriers) runs beside Z (the other seven), and the
// Cholesky factor and its inverse are one wave's too; lanes' values go through scalar registers.
// 512 x 20: 24 us (27 through LDS), with 256 threads and a barrier for each pivot and column 64 us.
// ls_apply_k takes 6.0 us where rows, rotation and copy took 17.7, ls_inv_k 8.9 (34 for the modes in
// turn).  Ten sweeps at 512^3, R = 20 (two on FP32 X), whole fit: 3.67 ms (6.11).
#include <algorithm>
#include <mutex>

#include "nnc_internal.h"

namespace nnc {

namespace {

constexpr int kLsThreads = 512;   // ls_small_k
constexpr int kLsChunk = 256;     // rows of num staged in LDS at a time (doubles, R <= 32: 64 KB)
constexpr int kLsSplit = 32;      // row ranges of Z at most

typedef double d2 __attribute__((ext_vector_type(2)));

// 1 / x and 1 / sqrt(x) by the hardware's estimates and two Newton steps (an ulp or two of double).
__device__ inline double rcp_d(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}
__device__ inline double rsqrt_d(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// A wave's own LDS exchange: what its lanes wrote is there for its next reads.
__device__ inline void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// x of lane k, in scalar registers: the exchanges below run without LDS, whose write, wait and
// broadcast reads were half of a pivot's time.
__device__ inline double lane_value(double x, int k) {
  const long long v = __double_as_longlong(x);
  const unsigned int lo = __builtin_amdgcn_readlane((int)v, k), hi = __builtin_amdgcn_readlane((int)(v >> 32), k);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Inverse of the r x r matrix whose row i lane i holds in a (r <= RM), by Gauss-Jordan elimination
// without pivoting, in place; every lane of one wave takes part.  Returns the number of pivots that
// are not positive.
template <int RM>
__device__ inline unsigned int wave_inverse(double (&a)[RM], int r, int lane) {
  unsigned int bad = 0;
#pragma unroll
  for (int k = 0; k < RM; ++k)
    if (k < r) {
      const double p = lane_value(a[k], k), ip = rcp_d(p);
      if (!(p > 0.0)) ++bad;
      const bool own = lane == k;
      const double f = own ? -ip : a[k] * ip;  // row k itself becomes row k / p
#pragma unroll
      for (int j = 0; j < RM; ++j)
        if (j != k) {
          const double v = lane_value(a[j], k);
          a[j] = fma(-f, v, own ? 0.0 : a[j]);
        }
      a[k] = -f;
    }
  return bad;
}

// Cholesky factor of the r x r matrix W (LDS, row stride RM) into L (row stride RM, zeros above the
// diagonal) and the inverse of L into Li, by one wave; lane i owns row i of L, then column i of Li.
// Returns the number of diagonal entries that are not positive.
template <int RM>
__device__ inline unsigned int wave_cholesky(const double *W, double *L, double *Li, int r, int lane) {
  unsigned int bad = 0;
  const int i0 = lane < r ? lane : 0;
  double a[RM], inv[RM];
#pragma unroll
  for (int j = 0; j < RM; ++j) a[j] = W[i0 * RM + j];
#pragma unroll
  for (int j = 0; j < RM; ++j) {
    inv[j] = 0.0;
    if (j < r) {
      const double d = lane_value(a[j], j);
      if (!(d > 0.0)) ++bad;
      inv[j] = rsqrt_d(d);
      const double l = lane >= j ? a[j] * inv[j] : 0.0, li = l * inv[j];
#pragma unroll
      for (int k = 0; k < RM; ++k)
        if (k > j) a[k] = fma(-li, lane_value(a[j], k), a[k]);  // lane k: L[k][j] / inv[j]
      a[j] = l;
    }
  }
  if (lane < r) {
#pragma unroll
    for (int j = 0; j < RM; ++j) L[lane * RM + j] = j < r ? a[j] : 0.0;
  }
  wave_fence();
  double x[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    x[i] = 0.0;
    if (i < r) {
      double v = i == lane ? 1.0 : 0.0;
#pragma unroll
      for (int k = 0; k < RM; ++k)
        if (k < i) v = fma(-L[i * RM + k], x[k], v);
      x[i] = v * inv[i];
    }
  }
  if (lane < r) {
#pragma unroll
    for (int i = 0; i < RM; ++i)
      if (i < r) Li[i * RM + lane] = x[i];
  }
  return bad;
}

// C = op(A) op(B) for r x r double matrices in LDS (row stride RM; op = transpose when ta / tb),
// one entry a thread, then a barrier.
template <int RM>
__device__ inline void small_mm(const double *A, bool ta, const double *B, bool tb, double *C, int r) {
  for (int e = threadIdx.x; e < RM * RM; e += blockDim.x) {
    const int i = e / RM, j = e % RM;
    if (i >= r || j >= r) continue;
    double v = 0.0;
#pragma unroll 4
    for (int k = 0; k < r; ++k) v = fma(A[ta ? k * RM + i : i * RM + k], B[tb ? j * RM + k : k * RM + j], v);
    C[e] = v;
  }
  __syncthreads();
}

// The R x R part of a factor step (see the top of the file), one workgroup.
//   num (N x R): the numerator rows; K (R x R): the system, or nullptr for the
//   orthonormalization of the factor given in num alone (K = I).
//   Writes T_out = K^{-1} L^{-T} (R x R doubles), L_out = L (R x R floats, upper triangle
//   zero) and S_out = T^T Z T (the Gram of the new factor).
template <int RM>
__global__ __launch_bounds__(kLsThreads) void ls_small_k(const float *__restrict__ num,
                                                         const float *__restrict__ K, int N, int R,
                                                         double *__restrict__ T_out, float *__restrict__ L_out,
                                                         float *__restrict__ S_out, unsigned long long *fails) {
  extern __shared__ __attribute__((aligned(16))) double sd[];
  __shared__ unsigned int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int P = RM * RM, H = RM / 2;
  double *Z = sd, *Kinv = sd + P, *W = sd + 2 * P, *L = sd + 3 * P, *Li = sd + 4 * P, *M = sd + 5 * P;
  double *rows = sd + 6 * P;  // kLsChunk x RM, zeros past R; then the ranges' sums of Z
  if (tid == 0) bad = 0;
  for (int e = tid; e < 6 * P; e += kLsThreads) sd[e] = 0.0;
  // Z = num^T num by blocks of 2 x 2 entries times row ranges, waves 1 and up; K^{-1} by wave 0
  const int zt = tid - 64, nb = H * H, split = min(kLsSplit, (kLsThreads - 64) / nb);
  const int zb = zt % nb, zs = zt / nb, zx = zb / H * 2, zy = zb % H * 2;
  const bool zon = zt >= 0 && zs < split;
  double z[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  for (int i0 = 0; i0 < N; i0 += kLsChunk) {
    const int nr = min(kLsChunk, N - i0), n = nr * RM;
    __syncthreads();  // the previous chunk has been used
    for (int e0 = tid; e0 < n; e0 += 8 * kLsThreads) {
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int e = e0 + k * kLsThreads, i = e / RM, c = e % RM;
        const bool ok = e < n && c < R;
        v[k] = num[ok ? (int64_t)(i0 + i) * R + c : 0];
        if (!ok) v[k] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (e0 + k * kLsThreads < n) rows[e0 + k * kLsThreads] = (double)v[k];
    }
    __syncthreads();
    if (zon) {
      const double *px = rows + zx, *py = rows + zy;
#pragma unroll 4
      for (int i = zs; i < nr; i += split) {
        const d2 x = *reinterpret_cast<const d2 *>(px + i * RM), y = *reinterpret_cast<const d2 *>(py + i * RM);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int q = 0; q < 2; ++q) z[p][q] = fma(x[p], y[q], z[p][q]);
      }
    } else if (i0 == 0 && wave == 0) {
      double a[RM];
#pragma unroll
      for (int j = 0; j < RM; ++j) a[j] = lane < R && j < R ? (K ? (double)K[lane * R + j] : (lane == j ? 1.0 : 0.0)) : 0.0;
      unsigned int nbad = 0;
      if (K) nbad = wave_inverse<RM>(a, R, lane);
      if (lane < R) {
#pragma unroll
        for (int j = 0; j < RM; ++j) Kinv[lane * RM + j] = a[j];
      }
      if (lane == 0 && nbad) atomicAdd(&bad, nbad);
    }
  }
  __syncthreads();
  if (zon) {
#pragma unroll
    for (int p = 0; p < 2; ++p) *reinterpret_cast<d2 *>(rows + zs * P + (zx + p) * RM + zy) = d2{z[p][0], z[p][1]};
  }
  __syncthreads();
  for (int e = tid; e < P; e += kLsThreads) {
    double v = 0.0;
    for (int s = 0; s < split; ++s) v += rows[s * P + e];
    Z[e] = v;
  }
  __syncthreads();
  small_mm<RM>(Z, false, Kinv, false, M, R);  // Z K^{-1}
  small_mm<RM>(Kinv, false, M, false, W, R);  // K^{-1} Z K^{-1} = A*^T A*
  if (wave == 0) {
    const unsigned int nbad = wave_cholesky<RM>(W, L, Li, R, lane);
    if (lane == 0 && nbad) atomicAdd(&bad, nbad);
  }
  __syncthreads();
  for (int e = tid; e < P; e += kLsThreads) {
    const int i = e / RM, j = e % RM;
    if (i < R && j < R) L_out[i * R + j] = (float)L[e];
  }
  small_mm<RM>(Kinv, false, Li, true, W, R);  // T = K^{-1} L^{-T}
  for (int e = tid; e < P; e += kLsThreads) {
    const int i = e / RM, j = e % RM;
    if (i < R && j < R) T_out[i * R + j] = W[e];
  }
  small_mm<RM>(Z, false, W, false, M, R);  // Z T
  small_mm<RM>(W, true, M, false, L, R);   // S = T^T (Z T)
  for (int e = tid; e < P; e += kLsThreads) {
    const int i = e / RM, j = e % RM;
    if (i < R && j < R) S_out[i * R + j] = (float)L[e];
  }
  if (tid == 0 && bad) atomicAdd(fails, (unsigned long long)bad);
}

// Blocks [0, row_blocks): A[i][c] = sum_s num[i][s] T[s][c] (FP64 sums), one thread per entry (num
// and A must not overlap).  The blocks after them: G <- G x_n L^T in place, a thread per line of
// mode n (pre x R x post): out[..i..] = sum_{l >= i} L[l][i] G[..l..].
template <int RM>
__global__ __launch_bounds__(256) void ls_apply_k(const float *__restrict__ num, const double *__restrict__ T, int N, int R,
                                                  float *__restrict__ A, int row_blocks, float *__restrict__ G,
                                                  const float *__restrict__ L, int64_t pre, int64_t post) {
  __shared__ double Ts[32 * 32];
  if ((int)blockIdx.x >= row_blocks) {
    float *Ls = reinterpret_cast<float *>(Ts);  // rows of RM, zeros past R
    for (int e = threadIdx.x; e < RM * RM; e += 256) {
      const int i = e / RM, c = e % RM;
      const float v = L[i < R && c < R ? i * R + c : 0];
      Ls[e] = i < R && c < R ? v : 0.f;
    }
    const int64_t t = (int64_t)((int)blockIdx.x - row_blocks) * 256 + threadIdx.x;
    const bool on = t < pre * post;
    const int64_t p = on ? t / post : 0, q = on ? t - p * post : 0;
    float *g = G + p * R * post + q;
    float x[RM];
#pragma unroll
    for (int l = 0; l < RM; ++l) x[l] = g[(l < R ? l : 0) * post];
    __syncthreads();
    if (!on) return;
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      float v = 0.f;
#pragma unroll
      for (int l = i; l < RM; ++l) v = fmaf(Ls[l * RM + i], x[l], v);  // zeros of L past R
      if (i < R) g[i * post] = v;
    }
    return;
  }
  for (int e0 = threadIdx.x; e0 < R * R; e0 += 4 * 256) {
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = e0 + k * 256 < R * R ? T[e0 + k * 256] : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (e0 + k * 256 < R * R) Ts[e0 + k * 256] = v[k];
  }
  __syncthreads();
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)N * R) return;
  const int64_t i = e / R;
  const int c = (int)(e - i * R);
  const float *x = num + i * R;
  double v = 0.0;
#pragma unroll 4
  for (int s = 0; s < R; ++s) v += (double)x[s] * Ts[s * R + c];
  A[e] = (float)v;
}

struct LsInvArgs {
  int d;
  int R[kMaxDim];
  const float *S[kMaxDim];
  float *Sinv[kMaxDim];
};

// Sinv[k] = S[k]^{-1} (as floats), one wave per mode.
template <int RM>
__global__ __launch_bounds__(64) void ls_inv_k(LsInvArgs g, unsigned long long *fails) {
  const float *S = g.S[0];
  float *Sinv = g.Sinv[0];
  int R = g.R[0];
#pragma unroll
  for (int k = 1; k < kMaxDim; ++k)
    if ((int)blockIdx.x == k) {
      S = g.S[k];
      Sinv = g.Sinv[k];
      R = g.R[k];
    }
  const int lane = threadIdx.x;
  double a[RM];
#pragma unroll
  for (int j = 0; j < RM; ++j) a[j] = lane < R && j < R ? (double)S[lane * R + j] : 0.0;
  const unsigned int bad = wave_inverse<RM>(a, R, lane);
  if (lane < R) {
#pragma unroll
    for (int j = 0; j < RM; ++j)
      if (j < R) Sinv[lane * R + j] = (float)a[j];
  }
  if (lane == 0 && bad) atomicAdd(fails, (unsigned long long)bad);
}

}  // namespace

static int ls_bound(int64_t R) { return R <= 8 ? 8 : (int)((R + 3) / 4 * 4); }

// LDS of ls_small_k: six R x R matrices and a chunk of rows or the ranges' sums of Z.
static size_t ls_small_lds(int RM) {
  const int split = std::min(kLsSplit, (kLsThreads - 64) / (RM / 2 * (RM / 2)));
  return sizeof(double) * (size_t)(6 * RM * RM + std::max(kLsChunk * RM, split * RM * RM));
}

nnc_status launch_ls_factor(const float *num, const float *K, int64_t N, int64_t R, float *A, double *T, float *Lf,
                            float *S_out, float *G, int64_t pre, int64_t post, unsigned long long *fails,
                            hipStream_t s) {
  if (R < 1 || R > 32) return fail(NNC_EUNSUPPORTED, "least-squares factor step: rank %lld outside 1..32", (long long)R);
  if (N < 1 || N * R > INT32_MAX) return fail(NNC_EUNSUPPORTED, "least-squares factor step: %lld rows", (long long)N);
  if (num == A) return fail(NNC_EINVAL, "least-squares factor step: num and A must differ");
  const int RM = ls_bound(R);
  const size_t lds = ls_small_lds(RM);
#define NNC_LS(RMV)                                                                                               \
  do {                                                                                                            \
    if (lds > 64 * 1024) {                                                                                        \
      static std::mutex mu;                                                                                       \
      static bool raised = false;                                                                                 \
      std::lock_guard<std::mutex> lk(mu);                                                                         \
      if (!raised) NNC_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(ls_small_k<RMV>),                   \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));            \
      raised = true;                                                                                              \
    }                                                                                                             \
    hipLaunchKernelGGL(ls_small_k<RMV>, dim3(1), dim3(kLsThreads), lds, s, num, K, (int)N, (int)R, T, Lf, S_out, fails); \
  } while (0)
  switch (RM) {
    case 8: NNC_LS(8); break;
    case 12: NNC_LS(12); break;
    case 16: NNC_LS(16); break;
    case 20: NNC_LS(20); break;
    case 24: NNC_LS(24); break;
    case 28: NNC_LS(28); break;
    default: NNC_LS(32);
  }
#undef NNC_LS
  const int64_t rb = (N * R + 255) / 256, gb = (pre * post + 255) / 256;
#define NNC_LSA(RMV)                                                                                                 \
  hipLaunchKernelGGL(ls_apply_k<RMV>, dim3((unsigned)(rb + gb)), dim3(256), 0, s, num, T, (int)N, (int)R, A, (int)rb, \
                     G, Lf, pre, post)
  if (RM <= 8)
    NNC_LSA(8);
  else if (RM <= 16)
    NNC_LSA(16);
  else if (RM <= 20)
    NNC_LSA(20);
  else
    NNC_LSA(32);
#undef NNC_LSA
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

nnc_status launch_ls_inverses(int d, const int64_t *R, float *const *S, float *const *Sinv,
                              unsigned long long *fails, hipStream_t s) {
  LsInvArgs a;
  a.d = d;
  int rmax = 1;
  for (int k = 0; k < kMaxDim; ++k) {
    a.R[k] = k < d ? (int)R[k] : 1;
    a.S[k] = k < d ? S[k] : nullptr;
    a.Sinv[k] = k < d ? Sinv[k] : nullptr;
    if (k < d) {
      if (R[k] < 1 || R[k] > 32)
        return fail(NNC_EUNSUPPORTED, "least-squares core step: rank %lld outside 1..32", (long long)R[k]);
      rmax = std::max(rmax, (int)R[k]);
    }
  }
#define NNC_LSI(RMV)                                                              \
  case RMV:                                                                       \
    hipLaunchKernelGGL(ls_inv_k<RMV>, dim3(d), dim3(64), 0, s, a, fails);         \
    break
  switch (ls_bound(rmax)) {
    NNC_LSI(8);
    NNC_LSI(12);
    NNC_LSI(16);
    NNC_LSI(20);
    NNC_LSI(24);
    NNC_LSI(28);
    NNC_LSI(32);
  }
#undef NNC_LSI
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc
