// HIP kernels for gfx950 (CDNA4): the contraction dispatcher, multiplicative update steps,
// residual reductions and conversions.
//
// Contraction forms (n-mode product with a transposed factor, Appendix A):
//   X viewed as [P][N][Q] (N = the contracted mode, Q = product of the later modes):
//     out[p][r][q] = sum_n F(n, r) * X[p][n][q].
// The matrix-core X-streaming kernels (pass_kernels.hip) take every shape with rank <= 32 and
// rows of at least one 16-byte chunk, but for short contracted indices in rows that are not whole
// chunks; the general kernel here takes the rest.
#include <stdarg.h>
#include <stdio.h>

#include <mutex>
#include <map>

#include <algorithm>

#include "nnc_internal.h"

namespace nnc {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

static __device__ inline uint16_t f2bf_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
static __device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

static __device__ inline float load_x(const float *p) { return *p; }
static __device__ inline float load_x(const uint16_t *p) { return bf2f(*p); }

static __device__ inline bf8 as_bf8(u4 v) { return __builtin_bit_cast(bf8, v); }

static __device__ inline f4 mfma_bf16(u4 a, u4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf8(a), as_bf8(b), c, 0, 0, 0);
}

// =====================================================================================
// General contraction (any shape, any R): one thread per (p, 4 columns r, q), sequential
// sum over the contracted index.
// =====================================================================================
template <typename XT>
__global__ __launch_bounds__(256) void ttm_generic_k(const XT *__restrict__ X, int64_t P, int64_t N,
                                                     int64_t Q, const float *__restrict__ F,
                                                     int64_t ldl, int64_t ldr, int64_t R,
                                                     float *__restrict__ out) {
  const int64_t RC = (R + 3) >> 2;
  const int64_t total = P * RC * Q;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = idx % Q;
    const int64_t t = idx / Q;
    const int64_t rc = t % RC;
    const int64_t p = t / RC;
    const int64_t r0 = rc * 4;
    const int nr = (int)((R - r0) < 4 ? (R - r0) : 4);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const XT *x = X + p * N * Q + q;
    for (int64_t l = 0; l < N; ++l) {
      const float xv = load_x(x + l * Q);
      const float *f = F + l * ldl + r0 * ldr;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < nr) acc[j] = fmaf(f[j * ldr], xv, acc[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < nr) out[(p * R + r0 + j) * Q + q] = acc[j];
  }
}

static int grid_for(int64_t work, int threads, int cap) {
  int64_t g = (work + threads - 1) / threads;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

nnc_status launch_ttm(const void *X, nnc_dtype xdt, int64_t P, int64_t N, int64_t Q, const float *F,
                      int64_t ldl, int64_t ldr, int64_t R, float *out, hipStream_t s,
                      bool allow_mfma, const char **kernel_name, int reserve_cus) {
  const char *name = "ttm_generic";
  const int64_t total_rows = P * N * Q;
  if (total_rows == 0 || R == 0) return NNC_OK;
  if (allow_mfma) {
    const nnc_status st = launch_pass(X, xdt, P, N, Q, F, ldl, ldr, R, out, s, kernel_name, reserve_cus);
    if (st != NNC_EUNSUPPORTED) return st;
  }
  // every other shape (rank above 32, rows shorter than 16 bytes, short ragged ones): one thread
  // per (p, 4 columns r, q)
  {
    const int64_t work = P * ((R + 3) / 4) * Q;
    const int grid = grid_for(work, 256, 65536);
    if (xdt == NNC_F32)
      hipLaunchKernelGGL(ttm_generic_k<float>, dim3(grid), dim3(256), 0, s, (const float *)X, P, N,
                         Q, F, ldl, ldr, R, out);
    else
      hipLaunchKernelGGL(ttm_generic_k<uint16_t>, dim3(grid), dim3(256), 0, s, (const uint16_t *)X,
                         P, N, Q, F, ldl, ldr, R, out);
  }
  if (kernel_name) *kernel_name = name;
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

// =====================================================================================
// Expansion of a rank mode to a data mode: out[p][n][q] = sum_r A[n][r] in[p][r][q], R <= 32
// (A row-major N x R), summed in rank order.  Bound by the write of out.
//   expand_wide_k  : long rows q: a thread keeps its column's R inputs (V adjacent columns) and
//                    walks a range of n, whose factor row is uniform over the block.
//   expand_short_k : short rows: out[p] is one contiguous block of N Q values; a thread keeps
//                    the factor row of its (n, q .. q + V - 1) and walks p, whose R x Q inputs
//                    pass through LDS a few p at a time.
// Measured (in brackets: the general contraction kernel, one thread per output column walking
// n): 64^4 x 8 from 64^3 x 8 x 8 111 us (560), 128^3 x 16 37 us (230), 256^2 x 32 16 us (26).
// The line between the two is where a row of q fills a block.
// =====================================================================================
template <int V>
struct ExpVec {
  float v[V];
};
template <int V>
static __device__ inline ExpVec<V> exp_load(const float *p) {
  ExpVec<V> x;
  if (V == 4) {
    const f4 y = *reinterpret_cast<const f4 *>(p);
#pragma unroll
    for (int i = 0; i < V; ++i) x.v[i] = y[i];
  } else {
    x.v[0] = *p;
  }
  return x;
}
template <int V>
static __device__ inline void exp_store(float *p, const ExpVec<V> &x) {
  if (V == 4)
    *reinterpret_cast<f4 *>(p) = f4{x.v[0], x.v[V > 1 ? 1 : 0], x.v[V > 2 ? 2 : 0], x.v[V > 3 ? 3 : 0]};
  else
    *p = x.v[0];
}

template <int RB, int V>
__global__ __launch_bounds__(256) void expand_wide_k(const float *__restrict__ in, int64_t P, int64_t R, int64_t Q,
                                                     const float *__restrict__ A, int64_t N, int64_t nper,
                                                     float *__restrict__ out) {
  const int64_t qv = Q / V;
  const int64_t n0 = blockIdx.y * nper, n1 = n0 + nper < N ? n0 + nper : N;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < P * qv; idx += (int64_t)gridDim.x * 256) {
    const int64_t p = idx / qv, q = (idx - p * qv) * V;
    ExpVec<V> x[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) x[r] = exp_load<V>(in + (p * R + (r < R ? r : 0)) * Q + q);
    for (int64_t n = n0; n < n1; ++n) {
      const float *a = A + n * R;
      ExpVec<V> acc;
#pragma unroll
      for (int i = 0; i < V; ++i) acc.v[i] = 0.f;
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (r < R) {
          const float f = a[r];
#pragma unroll
          for (int i = 0; i < V; ++i) acc.v[i] = fmaf(f, x[r].v[i], acc.v[i]);
        }
      exp_store<V>(out + (p * N + n) * Q + q, acc);
    }
  }
}

constexpr int kExpLds = 4096;  // floats of inputs staged at a time (whole p)

template <int RB, int V>
__global__ __launch_bounds__(256) void expand_short_k(const float *__restrict__ in, int64_t P, int R, int Q,
                                                      const float *__restrict__ A, int N, int64_t pper, int pb,
                                                      float *__restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) float xs[];
  const int nq = N * Q, rq = R * Q;
  const int e = (blockIdx.x * 256 + threadIdx.x) * V;
  const bool act = e < nq;
  const int n = act ? e / Q : 0, q = act ? e - n * Q : 0;
  float a[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) a[r] = r < R ? A[(int64_t)n * R + r] : 0.f;
  const int64_t p0 = blockIdx.y * pper, p1 = p0 + pper < P ? p0 + pper : P;
  for (int64_t pc = p0; pc < p1; pc += pb) {
    const int np = (int)(p1 - pc < pb ? p1 - pc : pb);
    __syncthreads();
    for (int x = threadIdx.x * V; x < np * rq; x += 256 * V) exp_store<V>(xs + x, exp_load<V>(in + pc * rq + x));
    __syncthreads();
    if (!act) continue;
    for (int j = 0; j < np; ++j) {
      ExpVec<V> acc;
#pragma unroll
      for (int i = 0; i < V; ++i) acc.v[i] = 0.f;
      const float *xp = xs + j * rq + q;
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (r < R) {
          const ExpVec<V> x = exp_load<V>(xp + r * Q);
#pragma unroll
          for (int i = 0; i < V; ++i) acc.v[i] = fmaf(a[r], x.v[i], acc.v[i]);
        }
      exp_store<V>(out + (pc + j) * nq + e, acc);
    }
  }
}

nnc_status launch_expand(const float *in, int64_t P, int64_t R, int64_t Q, const float *A, int64_t N, float *out,
                         hipStream_t s) {
  const bool v4 = Q % 4 == 0 && aligned16(in) && aligned16(out);
  const int64_t nq = N * Q;
  if (R > 32 || nq >= (1 << 24)) return launch_ttm(in, NNC_F32, P, R, Q, A, 1, R, N, out, s, false);
  if (Q >= 256 || R * Q > 2 * kExpLds) {
    const int64_t cols = P * (v4 ? Q / 4 : Q), bx = std::min<int64_t>((cols + 255) / 256, 65535);
    // ranges of n: enough blocks for the chip, at least 4 rows each
    const int64_t by = std::min<int64_t>(std::max<int64_t>(1, 2048 / bx), (N + 3) / 4), nper = (N + by - 1) / by;
#define NNC_EXP(RBV, VV)                                                                                     \
  hipLaunchKernelGGL((expand_wide_k<RBV, VV>), dim3((unsigned)bx, (unsigned)((N + nper - 1) / nper)), dim3(256), 0, \
                     s, in, P, R, Q, A, N, nper, out)
#define NNC_EXP_R(VV)          \
  do {                         \
    if (R <= 8)                \
      NNC_EXP(8, VV);          \
    else if (R <= 16)          \
      NNC_EXP(16, VV);         \
    else                       \
      NNC_EXP(32, VV);         \
  } while (0)
    if (v4)
      NNC_EXP_R(4);
    else
      NNC_EXP_R(1);
#undef NNC_EXP
  } else {
    const int64_t bx = (nq / (v4 ? 4 : 1) + 255) / 256;
    const int64_t by = std::min<int64_t>(std::max<int64_t>(1, 2048 / bx), P), pper = (P + by - 1) / by;
    const int pb = (int)std::min<int64_t>(std::max<int64_t>(1, kExpLds / (R * Q)), pper);
    const size_t lds = sizeof(float) * (size_t)(pb * R * Q);
#define NNC_EXP(RBV, VV)                                                                                      \
  hipLaunchKernelGGL((expand_short_k<RBV, VV>), dim3((unsigned)bx, (unsigned)((P + pper - 1) / pper)), dim3(256), lds, \
                     s, in, P, (int)R, (int)Q, A, (int)N, pper, pb, out)
    if (v4)
      NNC_EXP_R(4);
    else
      NNC_EXP_R(1);
#undef NNC_EXP
#undef NNC_EXP_R
  }
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

// =====================================================================================
// Small dense steps of the multiplicative updates.
// =====================================================================================
__global__ void contract_except_k(const float *__restrict__ U, const float *__restrict__ V,
                                  int64_t pre, int64_t I, int64_t J, int64_t post,
                                  float *__restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= I * J) return;
  const int64_t i = idx / J, j = idx - (idx / J) * J;
  float acc = 0.f;
  for (int64_t p = 0; p < pre; ++p) {
    const float *u = U + (p * I + i) * post;
    const float *v = V + (p * J + j) * post;
    for (int64_t q = 0; q < post; ++q) acc = fmaf(u[q], v[q], acc);
  }
  out[idx] = acc;
}

// The same contraction for J <= 32 on the FP32 matrix cores: a block takes 16 output rows, its
// eight waves one contiguous range each of the flattened summation index t = p * post + q, four
// values of t a step; the waves' sums are added in order through LDS.  Every value is read straight
// into the layout of the products, eight steps' loads together, so a block costs about two memory
// round trips (512 rows, t < 400, J = 20: 8.6 us; a wave per row with V in LDS and a butterfly per
// column: 17.5 us).  The eight steps of a round have an accumulator each, so a 64th of the products
// runs in order and the rest as a tree, as with a wave per row.
constexpr int kCeWaves = 8;

template <int RT, bool LONG>  // LONG: sums of 2^22 products and more, whose indices need the integer division
__global__ __launch_bounds__(64 * kCeWaves) void contract_except_rows_k(const float *__restrict__ U,
                                                                        const float *__restrict__ V, int pre,
                                                                        int64_t I, int J, int post,
                                                                        float *__restrict__ out) {
  __shared__ f4 part[kCeWaves][RT][64];
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (int64_t)blockIdx.x * 16;
  const int64_t ir = i0 + li < I ? i0 + li : I - 1;  // rows past I are computed and not stored
  const int total = pre * post, steps = (total + 3) >> 2, per = (steps + kCeWaves - 1) / kCeWaves;
  const int s1 = min(steps, (wave + 1) * per);
  const float inv_post = 1.0f / (float)post;
  int jc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) jc[rt] = min(16 * rt + li, J - 1);
  constexpr int kS = 8;
  f4 acc[kS][RT];
#pragma unroll
  for (int k = 0; k < kS; ++k)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[k][rt] = f4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = wave * per; s0 < s1; s0 += kS) {
    float u[kS], v[kS][RT];
#pragma unroll
    for (int k = 0; k < kS; ++k) {
      const int t = 4 * (s0 + k) + lg;
      const bool ok = s0 + k < s1 && t < total;
      const int tt = ok ? t : 0, p = LONG ? tt / post : qdiv(tt, inv_post), q = tt - p * post;
      u[k] = U[((int64_t)p * I + ir) * post + q];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) v[k][rt] = V[(p * J + jc[rt]) * post + q];
      if (!ok) {
        u[k] = 0.f;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) v[k][rt] = 0.f;
      }
    }
#pragma unroll
    for (int k = 0; k < kS; ++k)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        acc[k][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[k], v[k][rt], acc[k][rt], 0, 0, 0);
  }
  auto tree = [](const f4 (&x)[8]) { return ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7])); };
  static_assert(kS == 8 && kCeWaves == 8, "the trees below");
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    f4 x[kS];
#pragma unroll
    for (int k = 0; k < kS; ++k) x[k] = acc[k][rt];
    part[wave][rt][lane] = tree(x);
  }
  __syncthreads();
  if (wave >= RT) return;
  f4 x[kCeWaves];
#pragma unroll
  for (int w = 0; w < kCeWaves; ++w) x[w] = part[w][wave][lane];
  const f4 sum = tree(x);
  const int j = 16 * wave + li;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t i = i0 + 4 * lg + k;
    if (i < I && j < J) out[i * J + j] = sum[k];
  }
}

// The same contraction for few output rows (I small, J <= JM <= 32): one block of kSplitWaves
// waves per row i, wave w summing the contiguous range w of the flattened summation index
// (lanes striding inside it), a butterfly per wave, then the waves' sums added in wave order
// through LDS.
constexpr int kSplitWaves = 16;

template <int JM>
__global__ __launch_bounds__(64 * kSplitWaves) void contract_except_split_k(const float *__restrict__ U,
                                                                           const float *__restrict__ V,
                                                                           int pre, int64_t I, int J,
                                                                           int post,
                                                                           float *__restrict__ out) {
  __shared__ float ws[kSplitWaves][JM];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t i = blockIdx.x;
  const int total = pre * post;
  const int per = (total + kSplitWaves - 1) / kSplitWaves;
  const int tb = w * per, te = min(total, tb + per);
  float acc[JM];
#pragma unroll
  for (int j = 0; j < JM; ++j) acc[j] = 0.f;
  for (int t0 = tb + lane; t0 < te; t0 += 256) {
    float u[4];
    int vo[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int t = t0 + 64 * k;
      const bool ok = t < te;
      const int tt = ok ? t : tb;
      const int p = tt / post, q = tt - (tt / post) * post;
      u[k] = ok ? U[((int64_t)p * I + i) * post + q] : 0.f;
      vo[k] = p * J * post + q;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int j = 0; j < JM; ++j)
        if (j < J) acc[j] = fmaf(u[k], V[vo[k] + j * post], acc[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < JM; ++j) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) acc[j] += __shfl_xor(acc[j], m, 64);
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < JM; ++j) ws[w][j] = acc[j];
  }
  __syncthreads();
  if (threadIdx.x < J) {
    float sum = 0.f;
    for (int ww = 0; ww < kSplitWaves; ++ww) sum += ws[ww][threadIdx.x];
    out[i * J + threadIdx.x] = sum;
  }
}

nnc_status launch_contract_except(const float *U, const float *V, int64_t pre, int64_t I, int64_t J,
                                  int64_t post, float *out, hipStream_t s) {
  if (J <= 32 && I <= 64 && pre * post >= 64 * kSplitWaves && pre * J * post < INT32_MAX) {
    // few rows and a long sum: every row's sum split over a block of waves
#define NNC_CE_SPLIT(JM)                                                                        \
  hipLaunchKernelGGL(contract_except_split_k<JM>, dim3((unsigned)I), dim3(64 * kSplitWaves), 0, s, U, V, \
                     (int)pre, I, (int)J, (int)post, out)
    if (J <= 8)
      NNC_CE_SPLIT(8);
    else if (J <= 16)
      NNC_CE_SPLIT(16);
    else
      NNC_CE_SPLIT(32);
#undef NNC_CE_SPLIT
    NNC_HIP(hipGetLastError());
    return NNC_OK;
  }
  if (J <= 32 && pre * J * post < INT32_MAX && I < ((int64_t)1 << 31) / 64) {
    const int grid = (int)((I + 15) / 16);
#define NNC_CE_ROWS(RT, LONG)                                                                              \
  hipLaunchKernelGGL((contract_except_rows_k<RT, LONG>), dim3(grid), dim3(64 * kCeWaves), 0, s, U, V, (int)pre, I, \
                     (int)J, (int)post, out)
    if (pre * post < (1 << 22)) {
      if (J <= 16)
        NNC_CE_ROWS(1, false);
      else
        NNC_CE_ROWS(2, false);
    } else if (J <= 16) {
      NNC_CE_ROWS(1, true);
    } else {
      NNC_CE_ROWS(2, true);
    }
#undef NNC_CE_ROWS
    NNC_HIP(hipGetLastError());
    return NNC_OK;
  }
  const int64_t n = I * J;
  hipLaunchKernelGGL(contract_except_k, dim3(grid_for(n, 128, 1 << 30)), dim3(128), 0, s, U, V, pre,
                     I, J, post, out);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void gram_k(const float *__restrict__ A, int64_t N, int64_t R, float *__restrict__ S) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= R * R) return;
  const int64_t r = idx / R, c = idx - (idx / R) * R;
  float acc = 0.f;
  for (int64_t i = 0; i < N; ++i) acc = fmaf(A[i * R + r], A[i * R + c], acc);
  S[idx] = acc;
}

nnc_status launch_gram(const float *A, int64_t N, int64_t R, float *S, hipStream_t s) {
  if (R <= 32) return launch_gram_block(A, N, (int)R, S, s);  // one workgroup, rows staged in LDS
  hipLaunchKernelGGL(gram_k, dim3(grid_for(R * R, 64, 1 << 30)), dim3(64), 0, s, A, N, R, S);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

static __device__ inline float mu_step(float x, float num, float den, double eps,
                                       unsigned long long *clips) {
  double dd = (double)den;
  if (dd < eps) {
    dd = eps;
    atomicAdd(clips, 1ull);
  }
  return (float)(((double)x * (double)num) / dd);
}

// Rows are owned by one block; every thread reads its row of A before the barrier and
// writes its entry after it.
__global__ void mu_factor_k(float *__restrict__ A, const float *__restrict__ num,
                            const float *__restrict__ M, int64_t N, int64_t R, double eps,
                            unsigned long long *clips) {
  const int64_t rpb = blockDim.x / R;
  const int64_t i = (int64_t)blockIdx.x * rpb + threadIdx.x / R;
  const int64_t r = threadIdx.x % R;
  const bool act = threadIdx.x < rpb * R && i < N;
  float nv = 0.f;
  if (act) {
    float den = 0.f;
    for (int64_t s = 0; s < R; ++s) den = fmaf(A[i * R + s], M[s * R + r], den);
    nv = mu_step(A[i * R + r], num[i * R + r], den, eps, clips);
  }
  __syncthreads();
  if (act) A[i * R + r] = nv;
}

nnc_status launch_mu_factor(float *A, const float *num, const float *M, int64_t N, int64_t R,
                            double eps, unsigned long long *clips, hipStream_t s) {
  const int threads = 256;
  if (R > threads) return fail(NNC_EUNSUPPORTED, "rank %lld above %d", (long long)R, threads);
  const int64_t rpb = threads / R;
  hipLaunchKernelGGL(mu_factor_k, dim3((unsigned)((N + rpb - 1) / rpb)), dim3(threads), 0, s, A, num,
                     M, N, R, eps, clips);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void mu_elem_k(float *__restrict__ x, const float *__restrict__ num,
                          const float *__restrict__ den, int64_t n, double eps,
                          unsigned long long *clips) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = mu_step(x[i], num[i], den[i], eps, clips);
}

nnc_status launch_mu_elem(float *x, const float *num, const float *den, int64_t n, double eps,
                          unsigned long long *clips, hipStream_t s) {
  hipLaunchKernelGGL(mu_elem_k, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, x, num, den, n, eps,
                     clips);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void sub_k(const float *__restrict__ a, const float *__restrict__ b, float *__restrict__ o,
                      int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    o[i] = a[i] - b[i];
}

nnc_status launch_sub(const float *den, const float *num, float *out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(sub_k, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, den, num, out, n);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void matmul_small_k(const float *__restrict__ A, const float *__restrict__ M, int64_t N,
                               int64_t R, int64_t C, float *__restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= N * C) return;
  const int64_t i = idx / C, c = idx - (idx / C) * C;
  float acc = 0.f;
  for (int64_t s = 0; s < R; ++s) acc = fmaf(A[i * R + s], M[s * C + c], acc);
  out[idx] = acc;
}

nnc_status launch_matmul_small(const float *A, const float *M, int64_t N, int64_t R, int64_t C,
                               float *out, hipStream_t s) {
  hipLaunchKernelGGL(matmul_small_k, dim3(grid_for(N * C, 256, 1 << 30)), dim3(256), 0, s, A, M, N,
                     R, C, out);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

nnc_status launch_lift(const float *A, const float *B, int64_t N, int64_t Rm, int64_t r, float *C,
                       hipStream_t s) {
  return launch_matmul_small(A, B, N, Rm, r, C, s);
}

struct KrArgs {
  int d;
  int64_t dims[kMaxDim];
  const float *C[kMaxDim];
};

// W[m][rho] = prod_{k < d-1} C_k[i_k][rho] for the flattened leading index m.
__global__ void kr_rows_k(KrArgs a, int64_t lead, int64_t r, float *__restrict__ W) {
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < lead * r;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int64_t rho = idx % r;
    int64_t m = idx / r;
    float p = 1.f;
    for (int k = a.d - 2; k >= 0; --k) {
      const int64_t ik = m % a.dims[k];
      m /= a.dims[k];
      p *= a.C[k][ik * r + rho];
    }
    W[idx] = p;
  }
}

nnc_status launch_kr_rows(int d, const int64_t *dims, int64_t r, const float *const *C, float *W,
                          hipStream_t s) {
  KrArgs a;
  a.d = d;
  int64_t lead = 1;
  for (int k = 0; k < d; ++k) {
    a.dims[k] = dims[k];
    a.C[k] = C[k];
    if (k < d - 1) lead *= dims[k];
  }
  hipLaunchKernelGGL(kr_rows_k, dim3(grid_for(lead * r, 256, 65536)), dim3(256), 0, s, a, lead, r, W);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

// =====================================================================================
// Residual: sum over X (M x K) of (x - W[m,:] . Ad[k,:])^2 and of x^2, accumulated per
// thread in double, then a fixed-shape tree per block.  The grid size depends only on
// the problem size, so the summation order (and the result) is reproducible.
// =====================================================================================
constexpr int kResidThreads = 256;
constexpr int kResidMaxBlocks = 2048;

int resid_stream_max_blocks() { return kResidMaxBlocks; }

// ||X - Xhat||^2 and ||X||^2 with Xhat[m][k] = sum_r W[m][r] Ad[k][r] (X viewed as M x K,
// W the expansion of every mode but the last, Ad the last factor), R <= 32.
// A wave owns a stripe of 64 NS columns (NS adjacent columns a lane, their factor rows in
// registers for the whole stripe) and walks X's rows, 8 or 16 at a time with the next ones'
// loads in flight: X is read once in whole row segments, straight into the layout of its products.  Those run on the FP32 matrix cores
// as 4 x 4 x 1 blocks, one per four lanes: a block's four columns are its lanes', its four rows
// are X's, and W's 4 x 16 entries (four rows, sixteen ranks) sit in one register whose block r
// the instruction broadcasts to all (cbsz 4, abid r), so a row group costs R / 16 loads of W.
// Products add rank by rank in FP32, as a chain of fused multiply-adds would.  Each difference
// is formed and squared in FP64; sums are FP64 per lane, then per block.
// Bound: the read of X; the matrix cores need 8 R cycles per 64 NS x 4 entries, the FP64 side
// about 20 per 64.  Rows past M are read clamped and left out of the sums.
// Measured (in brackets: one thread per column with all ranks as VALU products, which left
// threads idle where K < 256): 64^5 FP32 at R = 8 892 us (2996), 128^4 BF16 at R = 16 176 us
// (488), 512^3 FP32 at R = 20 123 us (152), 256^3 FP32 at R = 32 29 us (59).
constexpr int kResidWaves = kResidThreads / 64;

// NS adjacent elements of X at any element boundary, as loaded, and as floats.
template <typename XT, int NS>
struct ResidRaw;
template <>
struct ResidRaw<float, 1> {
  static constexpr int kRows = 16;  // rows a wave loads at a time (one such tile is in flight
  float x;                          // while the one before is used)
  __device__ void load(const float *p) { x = *p; }
  __device__ float get(int) const { return x; }
};
template <>
struct ResidRaw<float, 2> {
  typedef float f2_el __attribute__((ext_vector_type(2), aligned(4)));
  static constexpr int kRows = 8;
  float x, y;
  __device__ void load(const float *p) {
    const f2_el v = *reinterpret_cast<const f2_el *>(p);
    x = v[0];
    y = v[1];
  }
  __device__ float get(int s) const { return s ? y : x; }
};
template <>
struct ResidRaw<uint16_t, 1> {
  static constexpr int kRows = 16;
  uint16_t x;
  __device__ void load(const uint16_t *p) { x = *p; }
  __device__ float get(int) const { return bf2f(x); }
};
template <>
struct ResidRaw<uint16_t, 2> {
  typedef uint32_t u1_el __attribute__((aligned(2)));
  static constexpr int kRows = 16;
  uint32_t x;
  __device__ void load(const uint16_t *p) { x = *reinterpret_cast<const u1_el *>(p); }
  __device__ float get(int s) const { return __uint_as_float(s ? x & 0xffff0000u : x << 16); }
};

template <int RB, int r>
struct ResidChain {
  template <int NS>
  static __device__ inline void run(const float (&w)[(RB + 15) / 16], const float (&b)[NS][RB], f4 (&acc)[NS]) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      acc[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[r / 16], b[s][r], acc[s], 4, r % 16, 0);
    if constexpr (r + 1 < RB) ResidChain<RB, r + 1>::template run<NS>(w, b, acc);
  }
};

// Waves per SIMD: 16 rows in flight (NS 1, and BF16) and the factor's values in 128 registers up to 16
// ranks or 32 values a lane, else in 168.
static constexpr int resid_waves(int rb, int ns) { return rb * ns > 32 || (ns == 1 && rb > 16) ? 3 : 4; }

// nst stripes; the grid's waves take stripe gw % nst and row tiles gw / nst, + rstep, ...
// of kRows rows, or, with more stripes than waves, stripes gw, gw + sstep, ... and every row.
template <typename XT, int RB, int NS>
__global__ __launch_bounds__(kResidThreads) __attribute__((amdgpu_waves_per_eu(resid_waves(RB, NS)))) void resid_stream_k(
    const XT *__restrict__ X, int64_t M, int64_t K, const float *__restrict__ W, const float *__restrict__ Ad, int R,
    double *__restrict__ part, int64_t nst, int64_t sstep, int64_t rstep) {
  __shared__ double s0[kResidThreads], s1[kResidThreads];
  constexpr int RH = (RB + 15) / 16;
  constexpr int kRows = ResidRaw<XT, NS>::kRows;
  const int t = threadIdx.x, lane = t & 63;
  const int64_t gw = (int64_t)blockIdx.x * kResidWaves + __builtin_amdgcn_readfirstlane(t >> 6);
  const int wrow = lane & 3, wr = lane >> 2;
  double sr = 0.0, sx = 0.0;
  const int64_t ntile = (M + kRows - 1) / kRows;
  const int64_t row0 = nst <= sstep ? gw / nst : 0;
  const int64_t st0 = nst <= sstep ? (row0 < rstep ? gw % nst : nst) : gw;
  for (int64_t st = st0; st < nst; st += sstep) {
    const int k = ((int)st * 64 + lane) * NS;
    // a lane whose columns reach past the row reads the row's last NS and drops what is not its own
    const unsigned kb = (unsigned)(k + NS <= (int)K ? k : (int)K - NS);
    const bool odd = NS == 2 && k == K - 1;
    float b[NS][RB];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int64_t kc = k + s < K ? k + s : (int64_t)K - 1;
      typedef float f4_el __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
      for (int r = 0; r < RB; r += 4) {  // four ranks a load: a load of 64 rows costs 64 requests
        if (r + 4 <= R) {
          const f4_el v = *reinterpret_cast<const f4_el *>(Ad + kc * R + r);
#pragma unroll
          for (int i = 0; i < 4; ++i) b[s][r + i] = v[i];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) b[s][r + i] = r + i < R ? Ad[kc * R + r + i] : 0.f;
        }
      }
    }
    double lr[NS], lx[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) lr[s] = lx[s] = 0.0;
    auto load = [&](int64_t tile, ResidRaw<XT, NS> (&xv)[kRows], float (&w)[kRows / 4][RH]) {
      const int64_t m0 = tile * kRows;
      const int left = (int)(M - m0 < kRows ? M - m0 : kRows) - 1;  // the tile's last row
      const XT *x0 = X + m0 * K;
      const float *wt = W + m0 * R;
#pragma unroll
      for (int row = 0; row < kRows; ++row) xv[row].load(x0 + (int64_t)(row < left ? row : left) * K + kb);
#pragma unroll
      for (int g = 0; g < kRows / 4; ++g) {
        const int m = 4 * g + wrow < left ? 4 * g + wrow : left;
#pragma unroll
        for (int h = 0; h < RH; ++h) w[g][h] = wt[m * R + (wr + 16 * h < R ? wr + 16 * h : 0)];
      }
    };
    auto use = [&](int64_t tile, const ResidRaw<XT, NS> (&xv)[kRows], const float (&w)[kRows / 4][RH]) {
      auto rows = [&](int n) {  // the tile's first n rows
#pragma unroll
        for (int g = 0; g < kRows / 4; ++g) {
          f4 acc[NS];
#pragma unroll
          for (int s = 0; s < NS; ++s) acc[s] = f4{0.f, 0.f, 0.f, 0.f};
          float wg[RH];
#pragma unroll
          for (int h = 0; h < RH; ++h) wg[h] = wr + 16 * h < R ? w[g][h] : 0.f;
          ResidChain<RB, 0>::template run<NS>(wg, b, acc);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (4 * g + i >= n) continue;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
              const float xf = odd ? xv[4 * g + i].get(NS - 1) : xv[4 * g + i].get(s);
              const double x = (double)xf, df = x - (double)acc[s][i];
              lr[s] += df * df;
              lx[s] += x * x;
            }
          }
        }
      };
      const int64_t n = M - tile * kRows;
      if (n >= kRows)
        rows(kRows);
      else
        rows((int)n);
    };
    // one tile's loads in flight while the one before is used; the loads past the last tile
    // read it again
    ResidRaw<XT, NS> x0[kRows], x1[kRows];
    float w0[kRows / 4][RH], w1[kRows / 4][RH];
    auto at = [&](int64_t tile) { return tile < ntile ? tile : ntile - 1; };
    load(at(row0), x0, w0);
    for (int64_t tile = row0; tile < ntile; tile += 2 * rstep) {
      load(at(tile + rstep), x1, w1);
      __builtin_amdgcn_sched_barrier(0);
      use(tile, x0, w0);
      __builtin_amdgcn_sched_barrier(0);
      if (tile + rstep >= ntile) break;
      load(at(tile + 2 * rstep), x0, w0);
      __builtin_amdgcn_sched_barrier(0);
      use(tile + rstep, x1, w1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (k + s < K) {
        sr += lr[s];
        sx += lx[s];
      }
  }
  s0[t] = sr;
  s1[t] = sx;
  __syncthreads();
  for (int w = kResidThreads / 2; w > 0; w >>= 1) {
    if (t < w) {
      s0[t] += s0[t + w];
      s1[t] += s1[t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    part[2 * blockIdx.x] = s0[0];
    part[2 * blockIdx.x + 1] = s1[0];
  }
}

// Any rank: one thread per element, the rank loop from global memory (L1/L2 hits).
template <typename XT>
__global__ __launch_bounds__(kResidThreads) void resid_any_k(const XT *__restrict__ X, int64_t M,
                                                             int64_t K, const float *__restrict__ W,
                                                             const float *__restrict__ Ad,
                                                             int64_t R, double *__restrict__ part) {
  __shared__ double s0[kResidThreads], s1[kResidThreads];
  double sr = 0.0, sx = 0.0;
  const int64_t total = M * K;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = e / K, k = e - (e / K) * K;
    const float *w = W + m * R;
    const float *a = Ad + k * R;
    float xh = 0.f;
    for (int64_t r = 0; r < R; ++r) xh = fmaf(w[r], a[r], xh);
    const float x = load_x(X + e);
    const double df = (double)x - (double)xh;
    sr += df * df;
    sx += (double)x * (double)x;
  }
  s0[threadIdx.x] = sr;
  s1[threadIdx.x] = sx;
  __syncthreads();
  for (int w = kResidThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s0[threadIdx.x] += s0[threadIdx.x + w];
      s1[threadIdx.x] += s1[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s0[0];
    part[2 * blockIdx.x + 1] = s1[0];
  }
}

nnc_status launch_resid_stream(const void *X, nnc_dtype xdt, int64_t M, int64_t K, const float *W,
                               const float *Ad, int64_t R, double *part, int *nblocks_out,
                               hipStream_t s) {
  if (R < 1) return fail(NNC_EINVAL, "residual: rank %lld", (long long)R);
  if (R > 32 || K >= (1 << 30)) {
    const int grid = grid_for(M * K, kResidThreads, kResidMaxBlocks);
    if (xdt == NNC_F32)
      hipLaunchKernelGGL(resid_any_k<float>, dim3(grid), dim3(kResidThreads), 0, s,
                         (const float *)X, M, K, W, Ad, R, part);
    else
      hipLaunchKernelGGL(resid_any_k<uint16_t>, dim3(grid), dim3(kResidThreads), 0, s,
                         (const uint16_t *)X, M, K, W, Ad, R, part);
    *nblocks_out = grid;
    NNC_HIP(hipGetLastError());
    return NNC_OK;
  }
  // NS = 2 columns a lane (wider loads, W's loads shared) unless that leaves half a stripe idle
  const int64_t half = (K + 63) / 64;
  const int NS = K >= 2 && (half % 2 == 0 || half > 8) ? 2 : 1;
  const int rows = xdt == NNC_F32 && NS == 2 ? 8 : 16;  // the kernel's kRows
  const int64_t ntile = (M + rows - 1) / rows, nst = NS == 2 ? (half + 1) / 2 : half;
  // as many waves as reside together: one round of equal shares (a CU has four SIMDs, a block four waves)
  const int64_t most = std::min<int64_t>((int64_t)device_cu_count() * resid_waves((int)(R + 3) / 4 * 4, NS), kResidMaxBlocks);
  const int grid = (int)std::min<int64_t>((ntile * nst + kResidWaves - 1) / kResidWaves, most);
  const int64_t waves = (int64_t)grid * kResidWaves;
  const int64_t rstep = nst <= waves ? waves / nst : 1, sstep = waves;
#define NNC_RES(XT, RBV)                                                                                      \
  do {                                                                                                        \
    if (NS == 1)                                                                                              \
      hipLaunchKernelGGL((resid_stream_k<XT, RBV, 1>), dim3(grid), dim3(kResidThreads), 0, s, (const XT *)X,  \
                         M, K, W, Ad, (int)R, part, nst, sstep, rstep);                                       \
    else                                                                                                      \
      hipLaunchKernelGGL((resid_stream_k<XT, RBV, 2>), dim3(grid), dim3(kResidThreads), 0, s, (const XT *)X,  \
                         M, K, W, Ad, (int)R, part, nst, sstep, rstep);                                       \
  } while (0)
#define NNC_RES2(XT)                    \
  do {                                  \
    switch ((R + 3) / 4) {              \
      case 1: NNC_RES(XT, 4); break;    \
      case 2: NNC_RES(XT, 8); break;    \
      case 3: NNC_RES(XT, 12); break;   \
      case 4: NNC_RES(XT, 16); break;   \
      case 5: NNC_RES(XT, 20); break;   \
      case 6: NNC_RES(XT, 24); break;   \
      case 7: NNC_RES(XT, 28); break;   \
      default: NNC_RES(XT, 32);         \
    }                                   \
  } while (0)
  if (xdt == NNC_F32)
    NNC_RES2(float);
  else
    NNC_RES2(uint16_t);
#undef NNC_RES2
#undef NNC_RES
  *nblocks_out = grid;
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void reduce_pairs_k(const double *__restrict__ part, int n, double *__restrict__ out) {
  __shared__ double s0[256], s1[256];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    a += part[2 * i];
    b += part[2 * i + 1];
  }
  s0[threadIdx.x] = a;
  s1[threadIdx.x] = b;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s0[threadIdx.x] += s0[threadIdx.x + w];
      s1[threadIdx.x] += s1[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = s0[0];
    out[1] = s1[0];
  }
}

nnc_status launch_reduce_pairs(const double *part, int n, double *out, hipStream_t s) {
  hipLaunchKernelGGL(reduce_pairs_k, dim3(1), dim3(256), 0, s, part, n, out);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void convert_bf16_k(const float *__restrict__ in, uint16_t *__restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = f2bf_rne(in[i]);
}

// =====================================================================================
// Counter-based SplitMix64 (Steele, Lea & Flood, OOPSLA 2014): element i of a stream with
// key K is mix64(K + (i + 1) * GAMMA), mix64 being SplitMix64's finaliser; a uniform double
// in [0, 1) is its top 53 bits times 2^-53.  Each element depends only on (K, i), so any
// slice of a stream is generated on its own, in any order.
// =====================================================================================
constexpr uint64_t kSmGamma = 0x9E3779B97F4A7C15ull;

static __host__ __device__ inline uint64_t sm_mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

uint64_t uniform_stream_key(uint64_t seed, uint64_t stream_id) {
  return sm_mix64(sm_mix64(seed + kSmGamma) ^ (stream_id * 0xD1B54A32D192ED03ull));
}

__global__ void fill_uniform_k(uint64_t key, int64_t offset, int64_t n, float *__restrict__ out32,
                               double *__restrict__ out64) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t z = sm_mix64(key + (uint64_t)(offset + i + 1) * kSmGamma);
    const double u = (double)(z >> 11) * 0x1.0p-53;  // exact: 53-bit integer times 2^-53
    if (out32)
      out32[i] = (float)u;  // round to nearest even
    else
      out64[i] = u;
  }
}

nnc_status launch_fill_uniform(uint64_t key, int64_t offset, int64_t n, float *out32, double *out64,
                               hipStream_t s) {
  hipLaunchKernelGGL(fill_uniform_k, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s, key, offset, n,
                     out32, out64);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

nnc_status launch_convert_bf16(const float *in, uint16_t *out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(convert_bf16_k, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, in, out, n);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void check_finite_k(const float *__restrict__ x, int64_t n, unsigned int *flag) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    if (!isfinite(x[i])) atomicOr(flag, 1u);
}

nnc_status launch_check_finite(const float *x, int64_t n, unsigned int *flag, hipStream_t s) {
  hipLaunchKernelGGL(check_finite_k, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, x, n, flag);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

__global__ void fill_u64_k(unsigned long long *x, int64_t n, unsigned long long v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = v;
}

__global__ void fill_f32_k(float *x, int64_t n, float v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = v;
}

nnc_status launch_fill_u64(unsigned long long *x, int64_t n, unsigned long long v, hipStream_t s) {
  hipLaunchKernelGGL(fill_u64_k, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, x, n, v);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

nnc_status launch_fill_f32(float *x, int64_t n, float v, hipStream_t s) {
  hipLaunchKernelGGL(fill_f32_k, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, x, n, v);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc
