// Nonnegative CP of a small tensor (the Tucker core) by multiplicative updates, one workgroup
// per fit, with the two large contractions of a sweep on the FP32 matrix cores.
//
// The modes are split into a left and a right group, 0 .. s-1 and s .. d-1 (at most three each),
// and the tensor is taken as the matrix T of pL rows and pR columns over the groups' indices:
//   V = T  KR(B_s .. B_{d-1})            (pL x r), from the factors the sweep starts with,
//   modes 0 .. s-1 updated from V:       M_n = sum over V's other modes, rank by rank,
//   U = T^t KR(B_0 .. B_{s-1})           (pR x r), from the new left factors,
//   modes s .. d-1 updated from U,
// with KR the Khatri-Rao product of a group's factors.  The modes are still updated in order
// 0 .. d-1 with the newest factors, so a sweep is the one of nncp_k (cp_kernels.hip); the work
// is 2 |T| r products and sums over arrays of pL r and pR r values.  (nncp_k contracts one mode
// of T and walks the result once per mode, multiplying d - 2 factor entries into every term: 158 us
// a sweep for 8^5 at rank 16, where the two products need 3.4 us of the matrix cores.)
//
// What bounds it: each step is a phase of one workgroup between barriers, with a few LDS round
// trips in it, so phases are few and short.
//   - T never passes through LDS.  Each wave keeps its fragments of T and of T^t in registers for
//     the whole fit (8 waves hold up to 32768 values in each layout), or, for larger tensors, streams them from the L2.
//   - Factors are double buffered (a sweep writes the other buffer), so nothing is copied.
//   - The Gram of an updated factor is one wave's matrix product beside the next phase's work,
//     and H_n = Hadamard of the other Grams is finished inside the update, which multiplies the
//     last Gram in.
// Sums run in a fixed order: results are reproducible and do not depend on what else is launched.
//
// Measured, us a sweep (nncp_k in brackets): 8^5 at rank 16 12.4 (155), 24^3 at rank 16 7.7 (11.8), 20^3
// at rank 10 5.8 (8.3), 10 x 10 x 11 x 10 at rank 8 6.5 (27), 4 x 8 x 12 x 16 at rank 10 8.3 (23) and 12^3
// at rank 6 4.0 (5.2); a call adds 60 to 90 us.  The two products of 8^5 take 6.0 and 5.2 thousand of
// its 30 thousand cycles (4.1 each is what the matrix cores need); the rest is twelve phases of 0.7 to
// 2.3 thousand, chains of a few LDS round trips and, in the updates, an FP64 division.  Sixteen waves
// were slower: every instruction of a phase then issues four times per SIMD.
#include <map>
#include <mutex>

#include "cpm_plan.h"
#include "nnc_internal.h"

namespace nnc {

typedef float f4 __attribute__((ext_vector_type(4)));

struct CpmPtrs {
  float *p[kMaxDim];
};

static __device__ inline f4 cpm_mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Fragment of T (TR: of T^t) for a unit: `step` of its range stands for four contracted indices,
// one per lane group.
template <bool TR>
static __device__ inline float cpm_frag(const float *__restrict__ T, const CpmArgs &a, const CpmProd &p, const CpmUnit &u,
                                        int step, int li, int lg) {
  const int row = 16 * u.t + li, k = 4 * (u.q * p.kper + step) + lg;
  const bool ok = u.q < p.split && step < p.kper && row < (TR ? a.pR : a.pL) && k < (TR ? a.pL : a.pR);
  const float x = T[ok ? (TR ? k * a.pR + row : row * a.pR + k) : 0];
  return ok ? x : 0.f;
}

// The same for step group g read from memory while it is used: element e of lane group lg stands
// for index 16 g + 4 lg + e of T's row (one 16-byte load a lane), 16 g + 4 e + lg of T^t's.
template <bool TR>
static __device__ inline void cpm_load(const float *__restrict__ T, const CpmArgs &a, const CpmProd &p, const CpmUnit &u,
                                       int g, int li, int lg, float *x) {
  if (TR) {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = cpm_frag<true>(T, a, p, u, 4 * g + e, li, lg);
    return;
  }
  typedef float f4_el __attribute__((ext_vector_type(4), aligned(4)));
  const int row = 16 * u.t + li, k0 = 4 * u.q * p.kper, k = k0 + 16 * g + 4 * lg;
  const int end = min(a.pR, k0 + 4 * p.kper);
  if (u.q < p.split && row < a.pL && k + 4 <= end) {
    const f4_el v = *reinterpret_cast<const f4_el *>(T + row * a.pR + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = u.q < p.split && row < a.pL && k + e < end;
      const float v = T[ok ? row * a.pR + k + e : 0];
      x[e] = ok ? v : 0.f;
    }
  }
}

// A wave's part in a product of one pass, fixed for the fit: its first unit's tile and range, the
// step groups, and (kr, out) where the lane reads KR's rows and writes its own.
struct CpmLane {
  int kr, out, left, step, gps, kper;  // left: rows of out from the first tile's first, step: rows
};                                     // from one slot's tile to the next
template <int RS, int NS>
static __device__ inline CpmLane cpm_lane(const CpmProd &p, int orows, int wave, int nw, int li, int lg) {
  const CpmUnit u = cpm_unit<NS>(p, wave, nw, 0, 0);
  const bool any = u.q < p.split;
  CpmLane l;
  l.kr = ((any ? 4 * u.q * p.kper : 0) + lg) * RS + li;
  l.out = (u.q * orows + 16 * u.t + 4 * lg) * RS + li;
  l.left = any ? orows - 16 * u.t : 0;
  l.step = 16 * nw;
  l.gps = any ? (p.kper + 3) >> 2 : 0;
  l.kper = p.kper;
  return l;
}

// A wave's fragments of T (or T^t), in the order cpm_product takes them.
template <int NS, int NR, bool TR>
static __device__ inline void cpm_frags(const float *__restrict__ T, const CpmArgs &a, const CpmProd &p, int wave, int nw,
                                        int li, int lg, float (&x)[NR]) {
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const CpmUnit u = cpm_unit<NS>(p, wave, nw, 0, s);
#pragma unroll
    for (int i = 0; i < NR / NS; ++i) x[(i / 4 * NS + s) * 4 + i % 4] = cpm_frag<TR>(T, a, p, u, i, li, lg);
  }
}

template <int RS, int RT>
static __device__ inline void cpm_write(float *o, const f4 (&acc)[RT], int left, int li, int lg) {
  const bool col = RS >= 16 || li < RS;
  if (left >= 16) {
    if (col) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j * RS + 16 * rt] = acc[rt][j];
    }
  } else {
    const int rows = col ? left - 4 * lg : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < rows) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) o[j * RS + 16 * rt] = acc[rt][j];
      }
  }
}

// out[range][row][c] = sum over the unit's range of T (or T^t) times KR (rows of RS), T's values
// in registers (x).  The operand rows of CH step groups are read together and their products follow
// in one block, so each waits for its own rows alone (T is zero past the range, whose rows may lie
// past KR).  One chain of products per tile, or four (by step) for a single tile: a product that
// waits for the one before takes about 100 cycles, an independent one 32.
template <int RS, int NS, int NR>
static __device__ inline void cpm_product(const CpmLane &l, const float (&x)[NR], const float *KR, float *out, int li, int lg) {
  constexpr int RT = RS > 16 ? 2 : 1, NA = NS == 1 ? 4 : NS, NGR = NR / (4 * NS), CH = NGR < 4 ? NGR : 4;
  f4 acc[NA][RT];
#pragma unroll
  for (int s = 0; s < NA; ++s)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[s][rt] = f4{0.f, 0.f, 0.f, 0.f};
  const float *kr = KR + l.kr;
#pragma unroll
  for (int c = 0; c < NGR; c += CH)
    if (c < l.gps) {
      float b[CH][4][RT];
#pragma unroll
      for (int i = 0; i < 4 * CH; ++i)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) b[i / 4][i % 4][rt] = kr[(4 * c + i) * 4 * RS + 16 * rt];
#pragma unroll
      for (int i = 0; i < 4 * CH; ++i) {
        if (NS == 1 || 4 * c + i < l.kper) {
#pragma unroll
          for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
              f4 &d = acc[NS == 1 ? i % 4 : s][rt];
              d = cpm_mfma(x[((c + i / 4) * NS + s) * 4 + i % 4], b[i / 4][i % 4][rt], d);
            }
        }
      }
    }
  if (NS == 1) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc[0][rt] = (acc[0][rt] + acc[1][rt]) + (acc[2][rt] + acc[3][rt]);
  }
  float *o = out + l.out;
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (l.left > s * l.step) cpm_write<RS, RT>(o + s * l.step * RS, acc[s], l.left - s * l.step, li, lg);
}

// The same with T read from the L2 while it is used, in as many passes as its tiles take.  The
// next step group's loads are in flight during the products of the current one.
template <int RS, int NS, bool TR>
static __device__ inline void cpm_product_stream(const float *__restrict__ T, const CpmArgs &a, const CpmProd &p,
                                                 const float *KR, float *out, int wave, int nw, int li, int lg) {
  constexpr int RT = RS > 16 ? 2 : 1, NA = NS == 1 ? 4 : NS;
  const int orows = TR ? a.pR : a.pL, krows = TR ? a.pL : a.pR, gps = (p.kper + 3) >> 2;
  for (int pass = 0; pass < p.passes; ++pass) {
    CpmUnit u[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) u[s] = cpm_unit<NS>(p, wave, nw, pass, s);
    if (u[0].q >= p.split) break;
    f4 acc[NA][RT];
#pragma unroll
    for (int s = 0; s < NA; ++s)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[s][rt] = f4{0.f, 0.f, 0.f, 0.f};
    float v[2][4 * NS], b[2][4][RT];
    const int kb = 4 * u[0].q * p.kper;
    auto load = [&](int g, float *w, float (&bb)[4][RT]) {
#pragma unroll
      for (int s = 0; s < NS; ++s) cpm_load<TR>(T, a, p, u[s], g, li, lg, w + 4 * s);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float *kr = KR + min(kb + 16 * g + (TR ? 4 * e + lg : 4 * lg + e), krows - 1) * RS + li;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) bb[e][rt] = kr[16 * rt];
      }
    };
    auto products = [&](const float *w, const float (&bb)[4][RT]) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            f4 &d = acc[NS == 1 ? e : s][rt];
            d = cpm_mfma(w[4 * s + e], bb[e][rt], d);
          }
    };
    load(0, v[0], b[0]);
    for (int g = 0; g < gps; g += 2) {
      load(g + 1, v[1], b[1]);
      products(v[0], b[0]);
      load(g + 2, v[0], b[0]);
      products(v[1], b[1]);
    }
    if (NS == 1) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[0][rt] = (acc[0][rt] + acc[1][rt]) + (acc[2][rt] + acc[3][rt]);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (u[s].q < p.split)
        cpm_write<RS, RT>(out + (u[s].q * orows + 16 * u[s].t + 4 * lg) * RS + li, acc[s], orows - 16 * u[s].t, li, lg);
  }
}

// W = B^t B (RS rows of WS) by one wave: B is n x RS, zeros up to a multiple of four rows.
template <int RS>
static __device__ inline void cpm_gram(const float *B, int n, float *W, int li, int lg) {
  constexpr int RT = RS > 16 ? 2 : 1;
  f4 acc[4][RT][RT];  // by step: independent chains
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int x = 0; x < RT; ++x)
#pragma unroll
      for (int y = 0; y < RT; ++y) acc[e][x][y] = f4{0.f, 0.f, 0.f, 0.f};
  const float *Bl = B + lg * RS + li;
  for (int k = 0; k < n; k += 16) {
    float v[4][RT];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) v[e][rt] = Bl[(k + 4 * e) * RS + 16 * rt];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + 4 * e < n) {  // the last step's rows past n are zeros
#pragma unroll
        for (int x = 0; x < RT; ++x)
#pragma unroll
          for (int y = 0; y < RT; ++y) acc[e][x][y] = cpm_mfma(v[e][x], v[e][y], acc[e][x][y]);
      }
  }
#pragma unroll
  for (int x = 0; x < RT; ++x)
#pragma unroll
    for (int y = 0; y < RT; ++y) acc[0][x][y] = (acc[0][x][y] + acc[1][x][y]) + (acc[2][x][y] + acc[3][x][y]);
  if (RS >= 16 || (li < RS && 4 * lg < RS)) {
#pragma unroll
    for (int x = 0; x < RT; ++x)
#pragma unroll
      for (int y = 0; y < RT; ++y)
#pragma unroll
        for (int j = 0; j < 4; ++j) W[(16 * x + 4 * lg + j) * (RS + 4) + 16 * y + li] = acc[0][x][y][j];
  }
}

template <int RS, int NS, int NR, int D>
__global__ __launch_bounds__(64 * kCpmWaves) void nncp_mm_k(const float *__restrict__ T, CpmArgs a, int rank0, CpmPtrs ptr0,
                                                  const int *__restrict__ ranks, float *const *__restrict__ fptrs,
                                                  int iters, double eps, double *__restrict__ resid,
                                                  unsigned long long *clips, int lds_floats) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ unsigned int nclip;
  constexpr int S = (D + 1) / 2;  // modes of the left group
  constexpr int Q4 = RS / 4, WS = RS + 4, RR = RS * WS;
  const int nq = ((ranks ? ranks[blockIdx.x] : rank0) + 3) >> 2;  // quads of columns in use
  const float inv_nq = 1.0f / (float)nq;
  const int b = blockIdx.x;
  const int r = ranks ? ranks[b] : rank0;
  const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 15, lg = lane >> 4;
  float *const sB = sm;  // factor k, buffer c: sB + c * BS + off[k]
  const int BS = a.sumdim * RS;
  int off[D];
  float inv_dim[D];
  {
    int o = 0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      inv_dim[k] = 1.0f / (float)a.dims[k];
      off[k] = o;
      o += ((a.dims[k] + 3) & ~3) * RS;
    }
  }
  float *const sW = sm + 2 * BS;
  float *const Hp = sW + D * RR;
  float *const part = Hp + RR;
  float *const KL = part + max(4 * nt, a.maxdim * RS);
  float *const KR = KL + (S > 1 ? a.pL * RS : 0);
  float *const VU = KR + (D - S > 1 ? a.pR * RS : 0);

  // ---- the fit's state: factors, T's fragments, Grams
  if (tid == 0) nclip = 0;
  for (int e = tid; e < lds_floats; e += nt) sm[e] = 0.f;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const float *src = ranks ? fptrs[(int64_t)b * D + k] : ptr0.p[k];
    for (int e = tid; e < a.dims[k] * RS; e += nt) {
      const int i = e / RS, c = e % RS;
      if (c < r) sB[off[k] + e] = src[i * r + c];
    }
  }
  float fv[NR > 0 ? NR : 1], fu[NR > 0 ? NR : 1];
  if constexpr (NR > 0) {
    cpm_frags<NS, NR, false>(T, a, a.v, wave, nw, li, lg, fv);
    cpm_frags<1, NR, true>(T, a, a.u, wave, nw, li, lg, fu);
  }
  const CpmLane lv = cpm_lane<RS, NS>(a.v, a.pL, wave, nw, li, lg), lu = cpm_lane<RS, 1>(a.u, a.pR, wave, nw, li, lg);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < D; ++k)
    if (wave == k % nw) cpm_gram<RS>(sB + off[k], a.dims[k], sW + k * RR, li, lg);
  __syncthreads();

  // Khatri-Rao product of modes F .. L of one buffer
  auto kr_rows = [&](auto F, auto L, const float *B, int rows, float *out) {
    for (int e = tid; e < rows * Q4; e += nt) {
      int rest = e / Q4;
      const int c = e % Q4 * 4;
      f4 v = f4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
      for (int k = L; k >= F; --k) {
        const int up = k > F ? qdiv(rest, inv_dim[k]) : 0, i = rest - up * a.dims[k];
        const f4 x = *reinterpret_cast<const f4 *>(B + off[k] + i * RS + c);
        v = k == L ? x : v * x;
        rest = up;
      }
      *reinterpret_cast<f4 *>(out + e * 4) = v;
    }
  };
  // H without the Gram of the mode updated before n (that one may be forming now): one wave's
  // work beside a phase's other work
  auto h_part = [&](auto N) {
    constexpr int n = N, pv = (N + D - 1) % D;
    if (wave != (nw > 1 ? nw - 2 : 0)) return;
#pragma unroll
    for (int e = 0; e < RR / 4; e += 64) {
      if (e + lane >= RR / 4) break;
      f4 h = f4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
      for (int k = 0; k < D; ++k)
        if (k != n && k != pv) h *= *reinterpret_cast<const f4 *>(sW + k * RR + (e + lane) * 4);
      *reinterpret_cast<f4 *>(Hp + (e + lane) * 4) = h;
    }
  };
  // (by the rank, not RS, which depends on the launch's other fits)
  auto m_split = [&](int In, int terms) {
    return cpm_sum_ranges(qdiv(64 * max(nw - 2, 1), 1.0f / (float)(In * nq)), terms);
  };
  // M_n's partial sums from V or U (rows: the group F .. L, row-major, `split` ranges to add), four
  // ranks a thread, in rows of the fit's own quads (ps floats: m_split's ranges then stay within part
  // whatever the launch's largest rank).  Bo: the sweep's old factors, Bn: its new ones.
  const int ps = 4 * nq;
  auto m_part = [&](auto N, auto F, auto L, const float *Bo, const float *Bn, int rows, int split) {
    // the group's other modes: xm (if there are two) outside ym
    constexpr int n = N, o1 = F != N ? int(F) : F + 1, o2 = o1 + 1 != N ? o1 + 1 : o1 + 2;
    constexpr int xm = o2 <= L ? o1 : -1, ym = o2 <= L ? o2 : o1, x0 = xm >= 0 ? xm : 0;
    auto stride = [&](int k) {
      int st = RS;
#pragma unroll
      for (int q = F; q <= L; ++q)
        if (q > k) st *= a.dims[q];
      return st;
    };
    const int In = a.dims[n], Y = a.dims[ym], terms = xm >= 0 ? a.dims[x0] * Y : Y;
    const int Sp = m_split(In, terms);
    const int gn = stride(n), gy = stride(ym), gx = xm >= 0 ? stride(xm) : 0;
    const float *By = (ym < n ? Bn : Bo) + off[ym], *Bx = (xm < n ? Bn : Bo) + off[x0];
    for (int w = tid; w < In * nq * Sp; w += nt) {
      const int is = qdiv(w, inv_nq), c = (w - is * nq) * 4, s = qdiv(is, inv_dim[n]), i = is - s * In;
      f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
      for (int t = s; t < terms; t += Sp) {
        int yi = t, at = i * gn + c;
        f4 bx;
        if (xm >= 0) {
          const int xi = qdiv(t, inv_dim[ym]);
          yi = t - xi * Y;
          at += xi * gx;
          bx = *reinterpret_cast<const f4 *>(Bx + xi * RS + c);
        }
        at += yi * gy;
        const f4 by = *reinterpret_cast<const f4 *>(By + yi * RS + c);
        f4 v = *reinterpret_cast<const f4 *>(VU + at);
        for (int q = 1; q < split; ++q) v += *reinterpret_cast<const f4 *>(VU + at + q * rows * RS);
        if (xm >= 0) v *= bx;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = fmaf(v[j], by[j], acc[j]);
      }
      *reinterpret_cast<f4 *>(part + (s * In + i) * ps + c) = acc;
    }
  };
  // B_n <- B_n * M / max(B_n H, eps) into the other buffer, one value a thread (B_n H on the
  // matrix cores, four values a lane, was 60 to 150 % slower: longer chains on fewer waves); M:
  // `split` arrays of In rows, `ms` floats apart.  H is symmetric, so its row c is read for column c.
  auto update = [&](auto N, const float *M, int split, int ms, const float *Bo, float *Bn) {
    constexpr int n = N, pv = (N + D - 1) % D;
    const int In = a.dims[n];
    const float *B = Bo + off[n];
    for (int e = tid; e < In * RS; e += nt) {
      const int i = e / RS, c = e % RS;
      if (c >= r) continue;
      const float *Wp = sW + pv * RR + c * WS, *Hc = Hp + c * WS, *Bi = B + i * RS;
      f4 d4 = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < RS; t += 4) {
        const f4 x = *reinterpret_cast<const f4 *>(Bi + t), h = *reinterpret_cast<const f4 *>(Hc + t),
                 w = *reinterpret_cast<const f4 *>(Wp + t);
#pragma unroll
        for (int j = 0; j < 4; ++j) d4[j] = fmaf(x[j], h[j] * w[j], d4[j]);
      }
      float m = 0.f;
#pragma unroll 4
      for (int q = 0; q < split; ++q) m += M[(q * In + i) * ms + c];
      double den = (double)((d4[0] + d4[1]) + (d4[2] + d4[3]));
      if (den < eps) {
        den = eps;
        atomicAdd(&nclip, 1u);
      }
      Bn[off[n] + e] = (float)(((double)Bi[c] * (double)m) / den);
    }
  };
  auto gram = [&](auto N, const float *B) {  // beside a phase's other work, on the last wave
    if (wave == nw - 1) cpm_gram<RS>(B + off[N], a.dims[N], sW + N * RR, li, lg);
  };
#define NNC_M(k) std::integral_constant<int, (k)>()
  for (int it = 0; it < iters; ++it) {
    float *Bo = sB + (it & 1) * BS, *Bn = sB + ((it & 1) ^ 1) * BS;
    // modes F .. L of a group from its contraction in VU, in order
    auto group = [&](auto F, auto L, int rows, int split) {
      auto mode = [&](auto N) {
        if constexpr (N > F) gram(NNC_M(N - 1), Bn);
        if (N == 0 && it) gram(NNC_M(D - 1), Bo);
        h_part(N);
        m_part(N, F, L, Bo, Bn, rows, split);
        __syncthreads();
        constexpr int o1 = F != N ? int(F) : F + 1, o2 = o1 + 1 != N ? o1 + 1 : o1 + 2;
        update(N, part, m_split(a.dims[N], o2 <= L ? a.dims[o1] * a.dims[o2 <= L ? o2 : 0] : a.dims[o1]), ps, Bo, Bn);
        __syncthreads();
      };
      if constexpr (F == L) {
        update(F, VU, split, RS, Bo, Bn);
        __syncthreads();
      } else {
        mode(F);
        mode(NNC_M(F + 1));
        if constexpr (F + 2 <= L) mode(NNC_M(F + 2));
      }
    };
    // ---- left group
    if (D - S > 1) {
      kr_rows(NNC_M(S), NNC_M(D - 1), Bo, a.pR, KR);
      __syncthreads();
    }
    if constexpr (NR > 0)
      cpm_product<RS, NS>(lv, fv, D - S > 1 ? KR : Bo + off[S], VU, li, lg);
    else
      cpm_product_stream<RS, NS, false>(T, a, a.v, D - S > 1 ? KR : Bo + off[S], VU, wave, nw, li, lg);
    if (S == 1) h_part(NNC_M(0));
    __syncthreads();
    group(NNC_M(0), NNC_M(S - 1), a.pL, a.v.split);
    // ---- right group
    gram(NNC_M(S - 1), Bn);
    if (S > 1) {
      kr_rows(NNC_M(0), NNC_M(S - 1), Bn, a.pL, KL);
      __syncthreads();
    }
    if constexpr (NR > 0)
      cpm_product<RS, 1>(lu, fu, S > 1 ? KL : Bn + off[0], VU, li, lg);
    else
      cpm_product_stream<RS, 1, true>(T, a, a.u, S > 1 ? KL : Bn + off[0], VU, wave, nw, li, lg);
    if (D - S == 1) h_part(NNC_M(D - 1));
    __syncthreads();
    group(NNC_M(S), NNC_M(D - 1), a.pR, a.u.split);
  }
  float *B = sB + (iters & 1) * BS;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    float *dst = ranks ? fptrs[(int64_t)b * D + k] : ptr0.p[k];
    for (int e = tid; e < a.dims[k] * RS; e += nt)
      if (e % RS < r) dst[e / RS * r + e % RS] = B[off[k] + e];
  }
  if (tid == 0 && nclip) atomicAdd(clips, (unsigned long long)nclip);

  if (resid) {  // ||T - KL KR^t|| / ||T||, FP64 sums, fixed tree
    const float *kl = S > 1 ? KL : B + off[0], *kr = D - S > 1 ? KR : B + off[S];
    if (S > 1) kr_rows(NNC_M(0), NNC_M(S - 1), B, a.pL, KL);
    if (D - S > 1) kr_rows(NNC_M(S), NNC_M(D - 1), B, a.pR, KR);
    __syncthreads();
    double sr = 0.0, sx = 0.0;
    const int tl = (a.pL + 15) >> 4, tr = (a.pR + 15) >> 4;
    for (int q = wave; q < tl * tr; q += nw) {
      const int o0 = 16 * (q / tr), c0 = 16 * (q % tr);
      f4 acc = f4{0.f, 0.f, 0.f, 0.f};
      const float *ap = kl + min(o0 + li, a.pL - 1) * RS, *bp = kr + min(c0 + li, a.pR - 1) * RS;
#pragma unroll
      for (int k = 0; k < RS; k += 4) acc = cpm_mfma(ap[k + lg], bp[k + lg], acc);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int o = o0 + 4 * lg + j, c = c0 + li;
        if (o < a.pL && c < a.pR) {
          const double x = T[o * a.pR + c], df = x - (double)acc[j];
          sr += df * df;
          sx += x * x;
        }
      }
    }
    double *red = reinterpret_cast<double *>(VU);
    red[tid] = sr;
    red[nt + tid] = sx;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
      if (tid < w && tid + w < nt) {
        red[tid] += red[tid + w];
        red[nt + tid] += red[nt + tid + w];
      }
      __syncthreads();
    }
    if (tid == 0) resid[b] = red[nt] > 0.0 ? sqrt(red[0] / red[nt]) : 0.0;
  }
#undef NNC_M
}

// ------------------------------------------------------------------ launch
bool nncp_mm_fits(const CpProblem &pb, int max_rank, int threads) {
  return cpm_fits(pb.d, pb.dims, pb.size, max_rank, threads);
}

static nnc_status cpm_allow_lds(const void *kern, int64_t bytes) {
  static std::mutex mu;
  static std::map<const void *, int64_t> done;
  if (bytes <= 64 * 1024) return NNC_OK;
  std::lock_guard<std::mutex> lk(mu);
  auto it = done.find(kern);
  if (it != done.end() && it->second >= bytes) return NNC_OK;
  NNC_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  done[kern] = bytes;
  return NNC_OK;
}

nnc_status launch_nncp_mm(const float *T, const CpProblem &pb, int nbatch, const int *d_ranks, int max_rank,
                          float *const *d_factor_ptrs, float *const *single_ptrs, int iters, double eps,
                          double *d_resid, unsigned long long *clips, int threads, hipStream_t s) {
  threads = std::min(threads, kCpmMaxThreads);
  if (!nncp_mm_fits(pb, max_rank, threads)) return fail(NNC_EUNSUPPORTED, "nnCP shape does not suit the matrix-core kernel");
  const CpmPlan pl = cpm_plan(pb.d, pb.dims, threads);
  const CpmArgs &a = pl.a;
  if (pl.ns > 1 && a.v.split > 1) return fail(NNC_EUNSUPPORTED, "nnCP: ranges with several slots");
  const int64_t lds = cpm_lds_floats(a, cpm_rs(max_rank), threads) * 4;
  CpmPtrs p0;
  for (int k = 0; k < kMaxDim; ++k) p0.p[k] = (single_ptrs && k < pb.d) ? single_ptrs[k] : nullptr;
#define NNC_CPM5(RSV, NSV, NRV, DV)                                                                                \
  do {                                                                                                             \
    NNC_TRY(cpm_allow_lds(reinterpret_cast<const void *>(nncp_mm_k<RSV, NSV, NRV, DV>), lds));                     \
    hipLaunchKernelGGL((nncp_mm_k<RSV, NSV, NRV, DV>), dim3(nbatch), dim3(threads), (size_t)lds, s, T, a, max_rank, \
                       p0, d_ranks, d_factor_ptrs, iters, eps, d_resid, clips, (int)(lds / 4));                    \
  } while (0)
#define NNC_CPM4(RSV, NSV, NRV)             \
  do {                                      \
    if (pb.d == 3)                          \
      NNC_CPM5(RSV, NSV, NRV, 3);           \
    else if (pb.d == 4)                     \
      NNC_CPM5(RSV, NSV, NRV, 4);           \
    else                                    \
      NNC_CPM5(RSV, NSV, NRV, 5);           \
  } while (0)
#define NNC_CPM3(RSV, NSV)     \
  do {                         \
    if (pl.nr == 32)           \
      NNC_CPM4(RSV, NSV, 32);  \
    else if (pl.nr == 64)      \
      NNC_CPM4(RSV, NSV, 64);  \
    else                       \
      NNC_CPM4(RSV, NSV, 0);   \
  } while (0)
#define NNC_CPM(RSV)          \
  do {                        \
    if (pl.ns == 8)           \
      NNC_CPM4(RSV, 8, 64);   \
    else if (pl.ns == 4)      \
      NNC_CPM3(RSV, 4);       \
    else                      \
      NNC_CPM3(RSV, 1);       \
  } while (0)
  if (max_rank <= 8)
    NNC_CPM(8);
  else if (max_rank <= 16)
    NNC_CPM(16);
  else
    NNC_CPM(32);
#undef NNC_CPM
#undef NNC_CPM3
#undef NNC_CPM4
#undef NNC_CPM5
  NNC_HIP(hipGetLastError());
  return NNC_OK;
}

}  // namespace nnc
