// The SH exponential as the projection of the pointwise exponential (the
// function-space quantity that the scaling and squaring scheme stands in for),
// taken with a fixed quadrature.  A selectable accuracy mode; it changes the
// result.
//
//   F = eps * pair * (sum of the sphere-chunk partials)   (as in the squaring path)
//   c = F_0 / sqrt(4 pi),  f_q = sum_{i >= 1} F_i y_i(w_q)
//   V = exp(c) sum_q w_q exp(f_q) y(w_q)
// over the product rule of degree 8n - 1: 4n Gauss-Legendre latitudes times 8n
// azimuths (j + 1/2) 2 pi / 8n.
//
// The sums over the nodes are separable.  Per latitude, f's Fourier
// coefficients come from a Legendre transform; an azimuth in the first quarter gives f at its four
// mirror images from four short sums (cosines and sines of even and odd order);
// the exponentials go back through the same two steps transposed.  At 8 bands
// and 2,048 nodes that is about 34,000 instructions per receiver, exponentials
// included, where the sums as dense products with the nodes' basis were 262,000
// multiply-adds on MFMA.
//
// Adjoint for Vbar: Fbar_0 = (sum_j Vbar_j V_j) / sqrt(4 pi) and, for i >= 1,
//   Fbar_i = exp(c) sum_q w_q exp(f_q) g_q y_i(w_q),  g_q = sum_j Vbar_j y_j(w_q),
// g by the same two steps as f; W = eps * pair * Fbar feeds the pair adjoint.
//
// Layout: one receiver per lane, the latitudes dealt to the eight waves of a
// block (four at 1 band), whose partial sums are added in wave order through
// LDS at the end.  F (and Vbar) stay in LDS for all waves, so that a wave's
// registers hold one latitude's coefficients and its 64 sums: 128 registers,
// four waves per SIMD, and two blocks fit a CU.  Bound by
// VALU issue, with 57 of the CUs holding two of the 313 blocks at 20,000
// receivers.  Measured there at 8 bands: forward 159 -> 33 us, adjoint 196 -> 45
// us, and the launches that built the nodes' basis and added partial sums (21
// us) are gone.
#pragma once

#include "shv_exp_impl.h"

namespace shv {

template <int NB>
struct QuadTab;
#define SHV_QTAB(n)                                                                                       \
  template <>                                                                                             \
  struct QuadTab<n> {                                                                                     \
    static __device__ __forceinline__ const float* rows() { return shv_quad_rows_##n; }                   \
    static __device__ __forceinline__ float w(int t) { return shv_quad_w_##n[t]; }                        \
    static __device__ __forceinline__ constexpr float cosm(int j, int m) { return shv_quad_cos_##n[j][m]; } \
    static __device__ __forceinline__ constexpr float sinm(int j, int m) { return shv_quad_sin_##n[j][m]; } \
  };
SHV_QTAB(1)
SHV_QTAB(2)
SHV_QTAB(3)
SHV_QTAB(4)
SHV_QTAB(5)
SHV_QTAB(6)
SHV_QTAB(7)
SHV_QTAB(8)
#undef SHV_QTAB

template <int NB>
struct Quad {
  static constexpr int N = NB * NB;
  static constexpr int LATS = 4 * NB;                     // latitudes
  static constexpr int QUARTER = 2 * NB;                  // azimuths in a quarter
  static constexpr int WAVES = LATS < 8 ? LATS : 8;       // per block of 64 receivers
  static constexpr int H = (N + 1) / 2;                   // coefficients per exchange of the waves' sums
};

template <int NB, bool ADJ>
struct QuadShared {
  union {
    struct {
      float F[NB * NB][64];            // scaled so that a row's entries give Fourier amplitudes of log2(e) f
      float G[ADJ ? NB * NB : 1][64];  // Vbar, likewise for g
    } in;
    float red[Quad<NB>::WAVES][Quad<NB>::H][64];
  };
  float c[64];
  float cb[Quad<NB>::WAVES][64];  // partial sums of Vbar . V
};

// Fourier amplitudes at sgn z of the function with coefficients e (in LDS).
template <int NB, bool MEAN>
__device__ __forceinline__ void quad_up(const float (*e)[64], int lane, const float* __restrict__ Q, float sgn,
                                        float (&A)[NB], float (&B)[NB]) {
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    float a[2] = {0.0f, 0.0f}, b[2] = {0.0f, 0.0f};  // even and odd l - m
#pragma unroll
    for (int l = m; l < NB; ++l) {
      if (l == 0 && !MEAN) continue;
      const int s = (l - m) & 1;
      const float t = Q[lat_at<NB>(m) + l - m];
      a[s] = fmaf(t, e[idx(l, m)][lane], a[s]);
      if (m > 0) b[s] = fmaf(t, e[idx(l, -m)][lane], b[s]);
    }
    A[m] = fmaf(sgn, a[1], a[0]);
    B[m] = fmaf(sgn, b[1], b[0]);
  }
}

// Values at azimuths phi, -phi, pi - phi, pi + phi, phi the quarter's j-th.
template <int NB>
__device__ __forceinline__ void quad_values(const float (&A)[NB], const float (&B)[NB], int j, float (&f)[4]) {
  float ce = A[0], co = 0.0f, se = 0.0f, so = 0.0f;  // cosines and sines of even and odd order
#pragma unroll
  for (int m = 1; m < NB; ++m) {
    const float c = QuadTab<NB>::cosm(j, m), s = QuadTab<NB>::sinm(j, m);
    if (m & 1) {
      co = m == 1 ? c * A[m] : fmaf(c, A[m], co);
      so = m == 1 ? s * B[m] : fmaf(s, B[m], so);
    } else {
      ce = fmaf(c, A[m], ce);
      se = m == 2 ? s * B[m] : fmaf(s, B[m], se);
    }
  }
  const float p = ce + co, q = so + se, r = ce - co, t = so - se;
  f[0] = p + q;
  f[1] = p - q;
  f[2] = r + t;
  f[3] = r - t;
}

// The transposed step: C_m += sum of cos(m phi) v, S_m += sum of sin(m phi) v over the four.
template <int NB>
__device__ __forceinline__ void quad_gather(const float (&v)[4], int j, float (&C)[NB], float (&S)[NB]) {
  const float p = v[0] + v[1], q = v[2] + v[3], r = v[0] - v[1], t = v[2] - v[3];
  const float ce = p + q, co = p - q, so = r + t, se = r - t;
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    if (m == 0) {
      C[0] += ce;
      continue;
    }
    C[m] = fmaf(QuadTab<NB>::cosm(j, m), (m & 1) ? co : ce, C[m]);
    S[m] = fmaf(QuadTab<NB>::sinm(j, m), (m & 1) ? so : se, S[m]);
  }
}

// acc += the transposed transform of one latitude's sums, times the nodes' weight.
template <int NB>
__device__ __forceinline__ void quad_down(const float* __restrict__ Q, float sgn, float w, const float (&C)[NB],
                                          const float (&S)[NB], float (&acc)[NB * NB]) {
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    const float ea = w * C[m], eb = w * S[m], oa = sgn * ea, ob = sgn * eb;
#pragma unroll
    for (int l = m; l < NB; ++l) {
      const float t = Q[lat_at<NB>(m) + l - m];
      const bool odd = ((l - m) & 1) != 0;
      acc[idx(l, m)] = fmaf(t, odd ? oa : ea, acc[idx(l, m)]);
      if (m > 0) acc[idx(l, -m)] = fmaf(t, odd ? ob : eb, acc[idx(l, -m)]);
    }
  }
}

// This wave's latitudes: acc = sum over their nodes of w exp(f) (ADJ: times g) times the rows.
template <int NB, bool ADJ>
__device__ __forceinline__ void quad_sums(const QuadShared<NB, ADJ>& sh, int wave, int lane, float (&acc)[NB * NB]) {
#pragma unroll
  for (int i = 0; i < NB * NB; ++i) acc[i] = 0.0f;
#pragma unroll 1
  for (int t = wave; t < Quad<NB>::LATS; t += Quad<NB>::WAVES) {
    asm volatile("" ::: "memory");  // F and Vbar are read again per latitude rather than held in registers
    const float* __restrict__ Q = QuadTab<NB>::rows() + (t >> 1) * Lat<NB>::QP;
    const float sgn = (t & 1) ? -1.0f : 1.0f;
    float A[NB], B[NB], X[NB], Y[NB], C[NB], S[NB];
    quad_up<NB, false>(sh.in.F, lane, Q, sgn, A, B);
    if constexpr (ADJ) quad_up<NB, true>(sh.in.G, lane, Q, sgn, X, Y);
#pragma unroll
    for (int m = 0; m < NB; ++m) C[m] = S[m] = 0.0f;
#pragma unroll
    for (int j = 0; j < Quad<NB>::QUARTER; ++j) {
      float f[4];
      quad_values<NB>(A, B, j, f);
#pragma unroll
      for (int x = 0; x < 4; ++x) f[x] = __builtin_amdgcn_exp2f(f[x]);
      if constexpr (ADJ) {
        float g[4];
        quad_values<NB>(X, Y, j, g);
#pragma unroll
        for (int x = 0; x < 4; ++x) f[x] *= g[x];
      }
      quad_gather<NB>(f, j, C, S);
    }
    quad_down<NB>(Q, sgn, QuadTab<NB>::w(t >> 1), C, S, acc);
  }
}

// The waves' sums added in wave order, half of the coefficients at a time;
// wave w hands rows w, w + WAVES, ... of a half to put(i, sum).
template <int NB, bool ADJ, class Put>
__device__ __forceinline__ void quad_reduce(QuadShared<NB, ADJ>& sh, int wave, int lane, const float (&acc)[NB * NB],
                                            Put put) {
  constexpr int N = NB * NB, H = Quad<NB>::H, W = Quad<NB>::WAVES;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();  // the inputs (h = 0) or the first half's sums (h = 1) have been read
#pragma unroll
    for (int i = h * H; i < N && i < (h + 1) * H; ++i) sh.red[wave][i - h * H][lane] = acc[i];
    __syncthreads();
    for (int i = h * H + wave; i < N && i < (h + 1) * H; i += W) {
      float v = sh.red[0][i - h * H][lane];
#pragma unroll
      for (int w = 1; w < W; ++w) v += sh.red[w][i - h * H][lane];
      put(i, v);
    }
  }
}

constexpr float kLog2e = 1.44269504088896341f;

// Forward: Fpart [nchunks][N][P] -> vis [N][P]; saved (may be NULL) <- F [N][P].
template <int NB>
__global__ __launch_bounds__(64 * Quad<NB>::WAVES, 4) void k_exp_quad_fwd(const float* __restrict__ Fpart, int nchunks,
                                                                          int64_t P, float eps,
                                                                          float* __restrict__ vis,
                                                                          float* __restrict__ saved) {
  constexpr int N = NB * NB, W = Quad<NB>::WAVES;
  __shared__ QuadShared<NB, false> sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t p = (int64_t)blockIdx.x * 64 + lane;
  const bool ok = p < P;
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
#pragma unroll 4
  for (int i = wave; i < N; i += W) {
    float v = Fpart[(int64_t)i * P + q];
    for (int c = 1; c < nchunks; ++c) v += Fpart[((int64_t)c * N + i) * P + q];
    v = (v * shv_coef_lam[i]) * eps;
    if (saved && ok) saved[(int64_t)i * P + p] = v;
    if (i == 0) sh.c[lane] = v * SHV_INV_SQRT_4PI;
    sh.in.F[i][lane] = v * (shv_coef_norm[i] * kLog2e);
  }
  __syncthreads();
  float acc[N];
  quad_sums<NB, false>(sh, wave, lane, acc);
  const float ec = expf(sh.c[lane]);
  quad_reduce<NB, false>(sh, wave, lane, acc, [&](int i, float v) {
    if (ok) vis[(int64_t)i * P + p] = ec * (shv_coef_norm[i] * v);
  });
}

// Adjoint: gV, vis, saved F [N][P] -> W = eps pair Fbar [N][P].
template <int NB>
__global__ __launch_bounds__(64 * Quad<NB>::WAVES, 4) void k_exp_quad_bwd(const float* __restrict__ gV,
                                                                          const float* __restrict__ vis,
                                                                          const float* __restrict__ saved, int64_t P,
                                                                          float eps, float* __restrict__ Wout) {
  constexpr int N = NB * NB, W = Quad<NB>::WAVES;
  __shared__ QuadShared<NB, true> sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t p = (int64_t)blockIdx.x * 64 + lane;
  const bool ok = p < P;
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  float part = 0.0f;
#pragma unroll 4
  for (int i = wave; i < N; i += W) {
    const float f = saved[(int64_t)i * P + q], g = gV[(int64_t)i * P + q];
    part = fmaf(g, vis[(int64_t)i * P + q], part);
    if (i == 0) sh.c[lane] = f * SHV_INV_SQRT_4PI;
    sh.in.F[i][lane] = f * (shv_coef_norm[i] * kLog2e);
    sh.in.G[i][lane] = g * shv_coef_norm[i];
  }
  sh.cb[wave][lane] = part;
  __syncthreads();
  float acc[N];
  quad_sums<NB, true>(sh, wave, lane, acc);
  const float ec = expf(sh.c[lane]);
  quad_reduce<NB, true>(sh, wave, lane, acc, [&](int i, float v) {
    if (!ok) return;
    float fb = ec * (shv_coef_norm[i] * v);
    if (i == 0) {
      float cbar = sh.cb[0][lane];
#pragma unroll
      for (int w = 1; w < W; ++w) cbar += sh.cb[w][lane];
      fb = cbar * SHV_INV_SQRT_4PI;
    }
    Wout[(int64_t)i * P + p] = eps * shv_coef_lam[i] * fb;
  });
}

template <int NB>
hipError_t exp_quad_fwd_nb(const float* Fpart, int nchunks, int64_t P, float eps, float* vis, float* saved,
                           hipStream_t st) {
  k_exp_quad_fwd<NB><<<(unsigned)pair_blocks(P), 64 * Quad<NB>::WAVES, 0, st>>>(Fpart, nchunks, P, eps, vis, saved);
  return hipGetLastError();
}

template <int NB>
hipError_t exp_quad_bwd_nb(const float* gV, const float* vis, const float* saved, int64_t P, float eps, float* W,
                           hipStream_t st) {
  k_exp_quad_bwd<NB><<<(unsigned)pair_blocks(P), 64 * Quad<NB>::WAVES, 0, st>>>(gV, vis, saved, P, eps, W);
  return hipGetLastError();
}

}  // namespace shv
