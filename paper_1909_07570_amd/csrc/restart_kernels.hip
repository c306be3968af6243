// Many complete nnCANDELINC fits of one small 3-way tensor from different random starts,
// one workgroup (one wave) per start with everything in LDS: the study of Section 4.2, which
// runs Algorithms 1 and 2 a thousand times on the 4x4x4 example with known nnCPD at several
// assumed multiranks and compares the distributions of relative error and mean congruence.
//
//   Algorithm 1: nnTucker (multirank m) by the blockwise multiplicative rule, nnCP of the
//                core (rank r), lift C_n = A_n B_n.
//   Algorithm 2: nnCP of X (rank r), NMF of each CP factor A_n ~ W_n H_n (m_n columns),
//                lift C_n = W_n H_n.
// Each fit runs a fixed number of sweeps.  Then ||X - cp(C)|| / ||X|| (FP64 sums) and, when
// the true factors are given, the mean congruence of the r rank-one terms of cp(C) with the
// true ones under the component matching that maximises it (Section 4.1 scoring).
//
// Every dimension, multirank and rank is <= kTinyDim = 8.  Every matrix is held as 8 x 8 and every
// tensor as 8 x 8 x 8 floats, zeros outside, so that a wave's lane is entry (lane / 8, lane % 8) of
// a matrix and indices need no division; loops run over the sizes' bounds KN, KM, KR (4 or 8 for
// the dimensions, the multirank and the rank, template parameters), where the zeros add nothing.
// What bounds it: one wave alone on its SIMD (1000 starts, 256 CUs), a chain of LDS round trips of
// about 100 cycles; each step issues all its reads before its products, tensors that stay fixed over
// a fit's sweeps sit in registers, and independent steps share a round trip (the three NMFs of an
// Algorithm 2 fit, with every size at most 4; the numerators' and denominators' contractions).
// With run-time sizes (a division per index, a wait per product) 1000 starts of Algorithm 2 on
// 4 x 4 x 4 took 2.21 ms for 200 + 200 sweeps, now 0.29 ms; every sum runs in the same order as
// then.
#include <string.h>

#include "nnc_internal.h"

namespace nnc {

constexpr int kTinyDim = 8;
constexpr int kTinyThreads = 64;
constexpr int kTinyCube = kTinyDim * kTinyDim * kTinyDim;
constexpr int kTinySq = kTinyDim * kTinyDim;

struct TinyArgs {
  const float *X;
  int N[3], M[3], r, alg, nres;
  int outer, inner;       // sweeps of the first (nnTucker / nnCP of X) and second fit
  const float *inits;     // per start, see tiny_init_floats()
  int64_t init_stride;    // floats per start
  const float *truth[3];  // N_n x r true factors, or null (no congruence)
  double eps;
  double *rel, *cong;     // [nres]
  float *fout;            // lifted factors of every start (nullable): [nres][N0 + N1 + N2][r]
  unsigned long long *clips;
};

struct TinyLds {
  float X[kTinyCube], G[kTinyCube], T0[kTinyCube], T1[kTinyCube], T2[kTinyCube], T3[kTinyCube];
  float A[3][kTinySq], B[3][kTinySq], E[3][kTinySq], S[3][kTinySq], SE[3][kTinySq], C[3][kTinySq];
  float Mm[kTinySq], cg[kTinySq];
  double red[2][kTinyThreads];
};

struct TinyCtx {
  int lane, row, col;
  double eps;
  unsigned int clips;
};

static __device__ inline void tsync() { __syncthreads(); }

// x * num / max(den, eps) where valid, 0 elsewhere
static __device__ inline float tiny_mu(TinyCtx &c, float x, float num, float den, bool valid) {
  double dd = (double)den;
  if (dd < c.eps) {
    dd = c.eps;
    if (valid) ++c.clips;
  }
  const float v = (float)(((double)x * (double)num) / dd);
  return valid ? v : 0.f;
}

// K consecutive floats from a 16-byte boundary.
template <int K>
static __device__ inline void tiny_row(const float *p, float (&v)[K]) {
#pragma unroll
  for (int k = 0; k < K; k += 4) {
    const float4 x = *reinterpret_cast<const float4 *>(p + k);
    v[k] = x.x;
    v[k + 1] = x.y;
    v[k + 2] = x.z;
    v[k + 3] = x.w;
  }
}

// Strides of the modes of an 8 x 8 x 8 tensor.
static __device__ constexpr int tiny_stride(int n) { return n == 0 ? 64 : (n == 1 ? 8 : 1); }

// Entry `lane` of A^T A, A with K rows.
template <int K>
static __device__ inline float tiny_gram(const TinyCtx &c, const float *A) {
  float x[K], y[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    x[i] = A[i * 8 + c.row];
    y[i] = A[i * 8 + c.col];
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < K; ++i) s = fmaf(x[i], y[i], s);
  return s;
}

// The entries (o0, o1, o2) < (B0, B1, B2) of `in` with mode NM contracted, in its L first indices,
// against F (entry [l][o_NM]): f(cube index, value), each entry by one lane.
template <int NM, int L, int B0, int B1, int B2, typename Fn>
static __device__ inline void tiny_ttm(const TinyCtx &c, const float *in, const float *F, Fn f) {
#pragma unroll
  for (int e = 0; e < B0 * B1 * B2; e += kTinyThreads) {
    const int o = e + c.lane, o2 = o % B2, o1 = o / B2 % B1, o0 = o / (B2 * B1);
    if (B0 * B1 * B2 < kTinyThreads && o0 >= B0) return;
    const int on = NM == 0 ? o0 : (NM == 1 ? o1 : o2);
    const float *src = in + o0 * 64 + o1 * 8 + o2 - on * tiny_stride(NM);
    float x[L], w[L], s = 0.f;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      x[l] = src[l * tiny_stride(NM)];
      w[l] = F[l * 8 + on];
    }
#pragma unroll
    for (int l = 0; l < L; ++l) s = fmaf(x[l], w[l], s);
    f(o0 * 64 + o1 * 8 + o2, s);
  }
}

// Entry (i, a) = (lane / 8, lane % 8) of the contraction of U and V over the modes but NM, K indices
// each.
template <int NM, int K>
static __device__ inline float tiny_contract_except(const TinyCtx &c, const float *U, const float *V) {
  constexpr int P = NM == 0 ? 1 : 0, Q = NM == 2 ? 1 : 2;
  const float *u = U + c.row * tiny_stride(NM), *v = V + c.col * tiny_stride(NM);
  float s = 0.f;
#pragma unroll
  for (int x = 0; x < K; ++x) {
    float p[K], q[K];
    if (Q == 2) {
      tiny_row<K>(u + x * tiny_stride(P), p);
      tiny_row<K>(v + x * tiny_stride(P), q);
    } else {
#pragma unroll
      for (int y = 0; y < K; ++y) {
        p[y] = u[x * tiny_stride(P) + y * tiny_stride(Q)];
        q[y] = v[x * tiny_stride(P) + y * tiny_stride(Q)];
      }
    }
#pragma unroll
    for (int y = 0; y < K; ++y) s = fmaf(p[y], q[y], s);
  }
  return s;
}

// Mode NM of a sweep of the blockwise nnTucker rule.
template <int NM, int KN, int KM>
static __device__ inline void tiny_tucker_mode(TinyCtx &c, TinyLds &L, const int *N, const int *M) {
  constexpr int K1 = NM == 0 ? 1 : 0, K2 = NM == 2 ? 1 : 2;
  auto to = [](float *out) { return [out](int at, float v) { out[at] = v; }; };
  // X x_{k != NM} A_k^T and G x_{k != NM} S_k side by side
  tiny_ttm<K1, KN, K1 == 0 ? KM : KN, K1 == 1 ? KM : KN, KN>(c, L.X, L.A[K1], to(L.T0));
  tiny_ttm<K1, KM, KM, KM, KM>(c, L.G, L.S[K1], to(L.T1));
  tsync();
  tiny_ttm<K2, KN, NM == 0 ? KN : KM, NM == 1 ? KN : KM, NM == 2 ? KN : KM>(c, L.T0, L.A[K2], to(L.T2));
  tiny_ttm<K2, KM, KM, KM, KM>(c, L.T1, L.S[K2], to(L.T3));
  tsync();
  const float num = tiny_contract_except<NM, KM>(c, L.T2, L.G);
  L.Mm[c.lane] = tiny_contract_except<NM, KM>(c, L.T3, L.G);
  tsync();
  float *A = L.A[NM];
  float m[KM], x[KM], den = 0.f;
  tiny_row<KM>(A + c.row * 8, x);
#pragma unroll
  for (int k = 0; k < KM; ++k) m[k] = L.Mm[k * 8 + c.col];
#pragma unroll
  for (int k = 0; k < KM; ++k) den = fmaf(x[k], m[k], den);
  const float v = tiny_mu(c, A[c.lane], num, den, c.row < N[NM] && c.col < M[NM]);
  tsync();
  A[c.lane] = v;
  tsync();
  L.S[NM][c.lane] = tiny_gram<KN>(c, A);
  tsync();
}

// One sweep of the blockwise nnTucker rule: factors 0, 1, 2, then the core.
template <int KN, int KM>
static __device__ inline void tiny_tucker_sweep(TinyCtx &c, TinyLds &L, const int *N, const int *M) {
  tiny_tucker_mode<0, KN, KM>(c, L, N, M);
  tiny_tucker_mode<1, KN, KM>(c, L, N, M);
  tiny_tucker_mode<2, KN, KM>(c, L, N, M);
  auto to = [](float *out) { return [out](int at, float v) { out[at] = v; }; };
  tiny_ttm<0, KN, KM, KN, KN>(c, L.X, L.A[0], to(L.T0));
  tiny_ttm<0, KM, KM, KM, KM>(c, L.G, L.S[0], to(L.T1));
  tsync();
  tiny_ttm<1, KN, KM, KM, KN>(c, L.T0, L.A[1], to(L.T2));
  tiny_ttm<1, KM, KM, KM, KM>(c, L.T1, L.S[1], to(L.T3));
  tsync();
  constexpr int kE = (KM * KM * KM + kTinyThreads - 1) / kTinyThreads;
  float num[kE], den[kE];
  int at[kE], k = 0;
  tiny_ttm<2, KN, KM, KM, KM>(c, L.T2, L.A[2], [&](int o, float v) {
    at[k] = o;
    num[k++] = v;
  });
  k = 0;
  tiny_ttm<2, KM, KM, KM, KM>(c, L.T3, L.S[2], [&](int, float v) { den[k++] = v; });
#pragma unroll
  for (int e = 0; e < kE; ++e) {
    const int o = at[e];
    L.G[o] = tiny_mu(c, L.G[o], num[e], den[e], o / 64 < M[0] && o / 8 % 8 < M[1] && o % 8 < M[2]);
  }
  tsync();
}

// T's K x K entries that lane (i, rho) sums for mode NM, in registers for the whole fit.
template <int NM, int K>
static __device__ inline void tiny_slab(const TinyCtx &c, const float *T, float (&t)[K][K]) {
  constexpr int P = NM == 0 ? 1 : 0, Q = NM == 2 ? 1 : 2;
#pragma unroll
  for (int x = 0; x < K; ++x)
#pragma unroll
    for (int y = 0; y < K; ++y) t[x][y] = T[c.row * tiny_stride(NM) + x * tiny_stride(P) + y * tiny_stride(Q)];
}

template <int NM, int K, int KR>
static __device__ inline void tiny_cp_mode(TinyCtx &c, TinyLds &L, const float (&t)[K][K], float (*F)[kTinySq], int n,
                                           int r) {
  constexpr int P = NM == 0 ? 1 : 0, Q = NM == 2 ? 1 : 2;
  float fp[K], fq[K], x[KR], sp[KR], sq[KR];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    fp[k] = F[P][k * 8 + c.col];
    fq[k] = F[Q][k * 8 + c.col];
  }
  tiny_row<KR>(F[NM] + c.row * 8, x);
  tiny_row<KR>(L.S[P] + c.col * 8, sp);
  tiny_row<KR>(L.S[Q] + c.col * 8, sq);
  const float old = F[NM][c.lane];
  float num = 0.f, den = 0.f;
#pragma unroll
  for (int a = 0; a < K; ++a)
#pragma unroll
    for (int b = 0; b < K; ++b) num = fmaf(t[a][b], fp[a] * fq[b], num);
#pragma unroll
  for (int a = 0; a < KR; ++a) den = fmaf(x[a], sp[a] * sq[a], den);
  const float v = tiny_mu(c, old, num, den, c.row < n && c.col < r);
  tsync();
  F[NM][c.lane] = v;
  tsync();
  L.S[NM][c.lane] = tiny_gram<K>(c, F[NM]);
  tsync();
}

// `iters` sweeps of the CP rule on the tensor T (sizes d <= K) with factors F and rank r <= KR.
template <int K, int KR>
static __device__ inline void tiny_cp_fit(TinyCtx &c, TinyLds &L, const float *T, const int *d, float (*F)[kTinySq], int r,
                                          int iters) {
  for (int n = 0; n < 3; ++n) L.S[n][c.lane] = tiny_gram<K>(c, F[n]);
  float t0[K][K], t1[K][K], t2[K][K];
  tiny_slab<0, K>(c, T, t0);
  tiny_slab<1, K>(c, T, t1);
  tiny_slab<2, K>(c, T, t2);
  tsync();
  for (int it = 0; it < iters; ++it) {
    tiny_cp_mode<0, K, KR>(c, L, t0, F, d[0], r);
    tiny_cp_mode<1, K, KR>(c, L, t1, F, d[1], r);
    tiny_cp_mode<2, K, KR>(c, L, t2, F, d[2], r);
  }
}

// One half of an NMF sweep: X <- X * (D Y) / max(X (Y^T Y), eps) for lane entry (row, col) of X
// (xr x m), D's row in registers (K entries), and the Gram of the new X (KX rows).
template <int K, int KX, int KM>
static __device__ inline void tiny_nmf_half(TinyCtx &c, const float (&dr)[K], float *X, const float *Y, const float *SY,
                                            float *SX, int row, int col, bool valid, bool active) {
  float y[K], x[KM], sy[KM];
#pragma unroll
  for (int k = 0; k < K; ++k) y[k] = Y[k * 8 + col];
  tiny_row<KM>(X + row * 8, x);
  tiny_row<KM>(SY + col * 8, sy);
  const float old = X[row * 8 + col];
  float num = 0.f, den = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) num = fmaf(dr[k], y[k], num);
#pragma unroll
  for (int k = 0; k < KM; ++k) den = fmaf(x[k], sy[k], den);
  const float v = tiny_mu(c, old, num, den, valid);
  tsync();
  if (active) X[row * 8 + col] = v;
  tsync();
  float g0[KX], g1[KX], s = 0.f;
#pragma unroll
  for (int i = 0; i < KX; ++i) {
    g0[i] = X[i * 8 + row];
    g1[i] = X[i * 8 + col];
  }
#pragma unroll
  for (int i = 0; i < KX; ++i) s = fmaf(g0[i], g1[i], s);
  if (active) SX[row * 8 + col] = s;
  tsync();
}

// The three NMFs L.A[n] ~ L.B[n] L.E[n]^T, `iters` sweeps: side by side, 16 lanes each, when every
// size is at most 4, else one after another.
template <int KN, int KM, int KR>
static __device__ inline void tiny_nmf_fits(TinyCtx &c, TinyLds &L, const int *N, const int *M, int r, int iters) {
  constexpr bool kSide = KN == 4 && KM == 4 && KR == 4;
  for (int n = 0; n < 3; ++n) {
    L.S[n][c.lane] = tiny_gram<KN>(c, L.B[n]);
    L.SE[n][c.lane] = tiny_gram<KR>(c, L.E[n]);
  }
  tsync();
  for (int n0 = 0; n0 < 3; n0 += kSide ? 3 : 1) {
    const bool active = !kSide || c.lane < 48;
    const int n = kSide ? (active ? c.lane >> 4 : 0) : n0;
    const int row = kSide ? (c.lane >> 2) & 3 : c.row, col = kSide ? c.lane & 3 : c.col;
    const bool w = active && row < N[n] && col < M[n], h = active && row < r && col < M[n];
    float dr[KR], dc[KN];
    tiny_row<KR>(L.A[n] + row * 8, dr);
#pragma unroll
    for (int i = 0; i < KN; ++i) dc[i] = L.A[n][i * 8 + row];
    for (int it = 0; it < iters; ++it) {
      tiny_nmf_half<KR, KN, KM>(c, dr, L.B[n], L.E[n], L.SE[n], L.S[n], row, col, w, active);
      tiny_nmf_half<KN, KR, KM>(c, dc, L.E[n], L.B[n], L.S[n], L.SE[n], row, col, h, active);
    }
  }
}

// C = P Q (P: N x K, Q: K x r, or Q^T given as r x K when qt).
static __device__ void tiny_lift(const TinyCtx &c, const float *P, const float *Q, int K, int qt, float *C) {
  float s = 0.f;
  for (int k = 0; k < K; ++k) s = fmaf(P[c.row * 8 + k], qt ? Q[c.col * 8 + k] : Q[k * 8 + c.col], s);
  C[c.lane] = s;
  tsync();
}

// rows x cols values at `in` (row-major), or their transpose, into an 8 x 8 matrix
static __device__ const float *tiny_in(const TinyCtx &c, const float *in, int rows, int cols, bool tr, float *out) {
  const int i = tr ? c.col : c.row, j = tr ? c.row : c.col;
  out[c.lane] = i < rows && j < cols ? in[i * cols + j] : 0.f;
  return in + rows * cols;
}
static __device__ const float *tiny_in3(const TinyCtx &c, const float *in, const int *d, float *out) {
  for (int o = c.lane; o < kTinyCube; o += kTinyThreads) {
    const int i0 = o / 64, i1 = o / 8 % 8, i2 = o % 8;
    out[o] = i0 < d[0] && i1 < d[1] && i2 < d[2] ? in[(i0 * d[1] + i1) * d[2] + i2] : 0.f;
  }
  return in + d[0] * d[1] * d[2];
}

template <int KN, int KM, int KR>
__global__ __launch_bounds__(kTinyThreads) __attribute__((amdgpu_waves_per_eu(1, 2))) void tiny_candelinc_k(TinyArgs a) {
  __shared__ __attribute__((aligned(16))) TinyLds L;
  const int start = blockIdx.x;
  TinyCtx c{(int)threadIdx.x, (int)threadIdx.x >> 3, (int)threadIdx.x & 7, a.eps, 0u};
  const int *N = a.N, *M = a.M;
  const int r = a.r;
  const int xs = N[0] * N[1] * N[2];
  tiny_in3(c, a.X, N, L.X);
  const float *in = a.inits + (int64_t)start * a.init_stride;
  // initial values, laid out as documented for tiny_init_floats()
  if (a.alg == 1) {
    for (int n = 0; n < 3; ++n) in = tiny_in(c, in, N[n], M[n], false, L.A[n]);
    in = tiny_in3(c, in, M, L.G);
    for (int n = 0; n < 3; ++n) in = tiny_in(c, in, M[n], r, false, L.B[n]);
  } else {
    for (int n = 0; n < 3; ++n) in = tiny_in(c, in, N[n], r, false, L.A[n]);
    for (int n = 0; n < 3; ++n) in = tiny_in(c, in, N[n], M[n], false, L.B[n]);
    for (int n = 0; n < 3; ++n) in = tiny_in(c, in, M[n], r, true, L.E[n]);  // H_n as the factor H^T
  }
  for (float *t : {L.T0, L.T1, L.T2, L.T3})
    for (int o = c.lane; o < kTinyCube; o += kTinyThreads) t[o] = 0.f;
  tsync();
  if (a.alg == 1) {
    for (int n = 0; n < 3; ++n) L.S[n][c.lane] = tiny_gram<KN>(c, L.A[n]);
    tsync();
    for (int t = 0; t < a.outer; ++t) tiny_tucker_sweep<KN, KM>(c, L, N, M);
    tiny_cp_fit<KM, KR>(c, L, L.G, M, L.B, r, a.inner);  // nnCP of the core
    for (int n = 0; n < 3; ++n) tiny_lift(c, L.A[n], L.B[n], M[n], 0, L.C[n]);
  } else {
    tiny_cp_fit<KN, KR>(c, L, L.X, N, L.A, r, a.outer);
    tiny_nmf_fits<KN, KM, KR>(c, L, N, M, r, a.inner);
    for (int n = 0; n < 3; ++n) tiny_lift(c, L.B[n], L.E[n], M[n], 1, L.C[n]);
  }
  // relative error of cp(C), FP64 sums
  double se = 0.0, sx = 0.0;
  for (int o = c.lane; o < xs; o += kTinyThreads) {
    const int i = o / (N[1] * N[2]), j = (o / N[2]) % N[1], k = o % N[2];
    float xh = 0.f;
    for (int rho = 0; rho < r; ++rho) xh = fmaf(L.C[0][i * 8 + rho] * L.C[1][j * 8 + rho], L.C[2][k * 8 + rho], xh);
    const float xv = L.X[i * 64 + j * 8 + k];
    const double dl = (double)xv - (double)xh;
    se += dl * dl;
    sx += (double)xv * (double)xv;
  }
  L.red[0][c.lane] = se;
  L.red[1][c.lane] = sx;
  // congruence of component rho with true component sigma: product over modes of cosines
  if (a.truth[0]) {
    for (int o = c.lane; o < r * r; o += kTinyThreads) {
      const int rho = o / r, sg = o % r;
      double prod = 1.0;
      for (int n = 0; n < 3; ++n) {
        double dot = 0.0, n1 = 0.0, n2 = 0.0;
        for (int i = 0; i < N[n]; ++i) {
          const double u = L.C[n][i * 8 + rho], v = a.truth[n][i * r + sg];
          dot += u * v;
          n1 += u * u;
          n2 += v * v;
        }
        prod *= (n1 > 0 && n2 > 0) ? dot / sqrt(n1 * n2) : 0.0;
      }
      L.cg[o] = (float)prod;
    }
  }
  tsync();
  if (c.lane == 0) {
    double e = 0.0, x = 0.0;
    for (int l = 0; l < kTinyThreads; ++l) {
      e += L.red[0][l];
      x += L.red[1][l];
    }
    a.rel[start] = x > 0 ? sqrt(e / x) : 0.0;
  }
  tsync();  // the residual sums are read before red[] is reused
  if (a.truth[0]) {  // best matching: every permutation of r components, lanes in turn
    int nperm = 1;
    for (int k = 2; k <= r; ++k) nperm *= k;
    double best = -1e300;
    for (int pidx = c.lane; pidx < nperm; pidx += kTinyThreads) {
      int avail[kTinyDim];
      for (int k = 0; k < r; ++k) avail[k] = k;
      int code = pidx, left = r;
      double s = 0.0;
      for (int rho = 0; rho < r; ++rho) {  // factorial-base digits pick the unused targets
        int f = 1;
        for (int k = 2; k < left; ++k) f *= k;
        const int dgt = code / f;
        code -= dgt * f;
        s += L.cg[rho * r + avail[dgt]];
        for (int k = dgt; k < left - 1; ++k) avail[k] = avail[k + 1];
        --left;
      }
      best = fmax(best, s / r);
    }
    L.red[0][c.lane] = best;
    tsync();
    if (c.lane == 0) {
      double b = -1e300;
      for (int l = 0; l < kTinyThreads; ++l) b = fmax(b, L.red[0][l]);
      a.cong[start] = b;
    }
  }
  if (a.fout) {
    float *out = a.fout + (int64_t)start * (N[0] + N[1] + N[2]) * r;
    for (int n = 0; n < 3; ++n) {
      for (int o = c.lane; o < N[n] * r; o += kTinyThreads) out[o] = L.C[n][o / r * 8 + o % r];
      out += N[n] * r;
    }
  }
  if (c.clips && a.clips) atomicAdd(a.clips, (unsigned long long)c.clips);
}

int64_t tiny_init_floats(int alg, const int *N, const int *M, int r) {
  int64_t s = 0;
  if (alg == 1) {
    for (int n = 0; n < 3; ++n) s += (int64_t)N[n] * M[n] + (int64_t)M[n] * r;
    s += (int64_t)M[0] * M[1] * M[2];
  } else {
    for (int n = 0; n < 3; ++n) s += (int64_t)N[n] * r + (int64_t)N[n] * M[n] + (int64_t)M[n] * r;
  }
  return s;
}

nnc_status launch_tiny_candelinc(const float *X, const int *N, const int *M, int r, int alg, int nres,
                                 int outer, int inner, const float *inits, const float *const *truth,
                                 double eps, double *rel, double *cong, float *fout,
                                 unsigned long long *clips, hipStream_t s) {
  TinyArgs a;
  memset(&a, 0, sizeof a);
  a.X = X;
  for (int n = 0; n < 3; ++n) {
    a.N[n] = N[n];
    a.M[n] = M[n];
    a.truth[n] = truth ? truth[n] : nullptr;
  }
  a.r = r;
  a.alg = alg;
  a.nres = nres;
  a.outer = outer;
  a.inner = inner;
  a.inits = inits;
  a.init_stride = tiny_init_floats(alg, N, M, r);
  a.eps = eps;
  a.rel = rel;
  a.cong = cong;
  a.fout = fout;
  a.clips = clips;
  auto wide = [](const int *d) { return d[0] > 4 || d[1] > 4 || d[2] > 4; };
  const int kind = (wide(N) ? 4 : 0) + (wide(M) ? 2 : 0) + (r > 4 ? 1 : 0);
#define NNC_TINY(K, NV, MV, RV)                                                                         \
  case K:                                                                                               \
    hipLaunchKernelGGL((tiny_candelinc_k<NV, MV, RV>), dim3(nres), dim3(kTinyThreads), 0, s, a);        \
    break
  switch (kind) {
    NNC_TINY(0, 4, 4, 4);
    NNC_TINY(1, 4, 4, 8);
    NNC_TINY(2, 4, 8, 4);
    NNC_TINY(3, 4, 8, 8);
    NNC_TINY(4, 8, 4, 4);
    NNC_TINY(5, 8, 4, 8);
    NNC_TINY(6, 8, 8, 4);
    NNC_TINY(7, 8, 8, 8);
  }
#undef NNC_TINY
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc

namespace nnc {

// Mean congruence of two rank-r CP models with factors P[n], Q[n] (dims[n] x r): the
// congruence of components rho and sigma is the product over modes of the cosines of their
// factor columns (FP64), and the score is the largest mean over the matchings of components
// (every permutation).  One workgroup; a zero column has cosine 0.
struct CongArgs {
  int d, r;
  int64_t dims[kMaxDim];
  const float *P[kMaxDim], *Q[kMaxDim];
  double *out;
};

__global__ __launch_bounds__(256) void congruence_k(CongArgs a) {
  __shared__ double cg[kTinyDim * kTinyDim];
  __shared__ double best[256];
  const int tid = threadIdx.x, r = a.r;
  if (tid < r * r) {
    const int rho = tid / r, sg = tid % r;
    double prod = 1.0;
    for (int n = 0; n < a.d; ++n) {
      double dot = 0.0, n1 = 0.0, n2 = 0.0;
      for (int64_t i = 0; i < a.dims[n]; ++i) {
        const double u = a.P[n][i * r + rho], v = a.Q[n][i * r + sg];
        dot += u * v;
        n1 += u * u;
        n2 += v * v;
      }
      prod *= (n1 > 0 && n2 > 0) ? dot / sqrt(n1 * n2) : 0.0;
    }
    cg[tid] = prod;
  }
  __syncthreads();
  int nperm = 1;
  for (int k = 2; k <= r; ++k) nperm *= k;
  double b = -1e300;
  for (int pidx = tid; pidx < nperm; pidx += 256) {
    int avail[kTinyDim];
    for (int k = 0; k < r; ++k) avail[k] = k;
    int code = pidx, left = r;
    double s = 0.0;
    for (int rho = 0; rho < r; ++rho) {  // factorial-base digits pick the unused targets
      int f = 1;
      for (int k = 2; k < left; ++k) f *= k;
      const int dgt = code / f;
      code -= dgt * f;
      s += cg[rho * r + avail[dgt]];
      for (int k = dgt; k < left - 1; ++k) avail[k] = avail[k + 1];
      --left;
    }
    b = fmax(b, s / r);
  }
  best[tid] = b;
  __syncthreads();
  if (tid == 0) {
    double m = -1e300;
    for (int t = 0; t < 256; ++t) m = fmax(m, best[t]);
    *a.out = m;
  }
}

nnc_status launch_congruence(int d, const int64_t *dims, int r, const float *const *P, const float *const *Q,
                             double *out, hipStream_t s) {
  CongArgs a;
  memset(&a, 0, sizeof a);
  a.d = d;
  a.r = r;
  for (int n = 0; n < d; ++n) {
    a.dims[n] = dims[n];
    a.P[n] = P[n];
    a.Q[n] = Q[n];
  }
  a.out = out;
  hipLaunchKernelGGL(congruence_k, dim3(1), dim3(256), 0, s, a);
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc
