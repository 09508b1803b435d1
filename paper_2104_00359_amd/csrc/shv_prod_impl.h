// Visibility as the direct product chain of Eq. 12, and its adjoint.
//
// V = V'_1 * V'_2 * ... * V'_S: truncated SH products (Eqs. 6-7) of the
// projected floored blockers V'_i (Eq. 13), taken left to right in sphere
// order (truncated products are not associative, so the order is part of the
// result).  With h_i = PAIR (.) F'_i, the pair's log-cap vector without the
// factor eps (F'_i exactly as the pair kernels form it), V'_i has the
// coefficients sqrt(4 pi) e_0 + beta h_i with beta = 1 - e^-eps.  A product
// with the constant 1 is exact under truncation, so each step is
//   V <- V + beta (V * h_i),        starting from V = sqrt(4 pi) e_0.
// The adjoint of one step, with Vb the cotangent of its output:
//   hbar_i = beta (Vb * V_in),      Vb_in = Vb + beta (Vb * h_i)
// (the triple-product tensor is symmetric in its three indices).  hbar_i
// becomes the pair weights W_lm = PAIR_lm hbar_lm of the pair adjoint.
//
// From 6 bands up the products are taken in the sphere's frame (below); up to
// 5 bands as follows.
//
// The generated adjoint of the squaring computes 2 (a * b) for any a and b,
// output group by output group; one step costs one such product forward and
// two in the adjoint.  The chain is sequential in the spheres, so the
// parallelism is over receivers only.
//
// Layout: four waves per 64 receivers, wave G owning output group G of each
// product; the full vectors are exchanged through LDS once per sphere, in
// double buffers, one barrier per sphere.  Every wave forms the blocker
// vector h_i itself (a few hundred flops against a quarter of a product).
// The forward can record each step's input V_in, [S][N][P]; the adjoint reads
// them back in reverse, one sphere ahead.  The pair adjoint is linear in its
// weights, so each wave runs it on its own output group's share of hbar and
// writes its own sphere-gradient partial (rows (block, wave), reduced in
// order afterwards); only the two vectors cross LDS, which keeps a block's
// LDS small enough for two blocks per CU.

#pragma once

#include <cmath>
#include <type_traits>

#include "shv_exp_impl.h"
#include "shv_pair_impl.h"

namespace shv {

// h = PAIR (.) F' of one pair: the same rows and products as the pair forward
// kernel, each coefficient scaled by its PAIR[l][|m|].
template <int NB>
__device__ __forceinline__ void blocker_vec(const PairGeom& G, float (&h)[NB * NB]) {
  float g[NB], C[NB], Sn[NB], r[2][NB];
  cap_terms<NB>(G.t, G.u, G.s2, g);
  cs_powers<NB>(G.x, G.y, C, Sn);
  legendre_monic<NB>(G.z, r[0]);
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    if (m >= 1) legendre_row<NB>(m, G.z, 1.0f, r[(m - 1) & 1], r[m & 1]);
#pragma unroll
    for (int l = m; l < NB; ++l) {
      const float u = l == m ? g[l] : g[l] * r[m & 1][l];
      if (m == 0) {
        h[idx(l, 0)] = SHV_PAIR[l][0] * u;
      } else {
        h[idx(l, m)] = SHV_PAIR[l][m] * (u * C[m]);
        h[idx(l, -m)] = SHV_PAIR[l][m] * (u * Sn[m]);
      }
    }
  }
}

template <int NB>
struct ProdFwdShared {
  float X[2][NB * NB][64];
};

template <int NB, int G>
__device__ __forceinline__ void prod_fwd_group(float (*X)[NB * NB][64], int lane, int64_t p, bool ok,
                                               const float* __restrict__ pts, int64_t P,
                                               const float4* __restrict__ sph, int S, float hbeta,
                                               float* __restrict__ vis, float* __restrict__ states) {
  constexpr int N = NB * NB;
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  const float px = sel0(ok, pts[q]);
  const float py = sel0(ok, pts[P + q]);
  const float pz = sel0(ok, pts[2 * P + q]);
  float V[N];
#pragma unroll
  for (int i = 0; i < N; ++i) V[i] = i == 0 ? SHV_SQRT_4PI : 0.0f;
  for (int s = 0; s < S; ++s) {
    if (states && ok) {
      float* dst = states + (int64_t)s * N * P + p;
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (group_of<NB>(i) == G) dst[(int64_t)i * P] = V[i];
    }
    float h[N], T[N];
    blocker_vec<NB>(pair_geom(px, py, pz, sph[s]), h);
    SqGroup<NB, G>::adj(V, h, T);  // group G of 2 (V * h)
    const int b = s & 1;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (group_of<NB>(i) == G) X[b][i][lane] = fmaf(hbeta, T[i], V[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) V[i] = X[b][i][lane];
  }
  if (vis && ok) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (group_of<NB>(i) == G) vis[(int64_t)i * P + p] = V[i];
  }
}

// hbeta = beta / 2 (the generated product returns twice the product).
template <int NB>
__global__ __launch_bounds__(SHV_BLOCK) void k_prod_fwd(const float* __restrict__ pts, int64_t P,
                                                        const float4* __restrict__ sph, int S, float hbeta,
                                                        float* __restrict__ vis, float* __restrict__ states) {
  __shared__ ProdFwdShared<NB> sh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t p = (int64_t)blockIdx.x * 64 + lane;
  const bool ok = p < P;
  switch (wave) {
    case 0: prod_fwd_group<NB, 0>(sh.X, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
    case 1: prod_fwd_group<NB, 1>(sh.X, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
    case 2: prod_fwd_group<NB, 2>(sh.X, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
    default: prod_fwd_group<NB, 3>(sh.X, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
  }
}

template <int NB>
struct ProdBwdShared {
  float Vb[2][NB * NB][64];  // cotangent of the chain state
  float Vi[2][NB * NB][64];  // the current step's input V_in
  float gp[3][3][64];        // receiver-gradient partials of waves 1..3
};

template <int NB, int G>
__device__ __forceinline__ void prod_bwd_group(ProdBwdShared<NB>& sh, int lane, int64_t bx, int64_t p, bool ok,
                                               const float* __restrict__ gvis, const float* __restrict__ states,
                                               const float* __restrict__ pts, int64_t P,
                                               const float4* __restrict__ sph, int S, float hbeta,
                                               float* __restrict__ gpts, float4* __restrict__ gs_part) {
  constexpr int N = NB * NB;
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  const float px = sel0(ok, pts[q]);
  const float py = sel0(ok, pts[P + q]);
  const float pz = sel0(ok, pts[2 * P + q]);
  float gpx = 0.0f, gpy = 0.0f, gpz = 0.0f;
  float4* gs_row = gs_part + (bx * 4 + G) * S;
  // Cotangent of the chain's output (zero on tail lanes, so they add nothing
  // to the sphere sums), the input of the last step, and the next one ahead.
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (group_of<NB>(i) == G) sh.Vb[S & 1][i][lane] = sel0(ok, gvis[(int64_t)i * P + q]);
  float pre[N];
  if (S > 0) {
    const float* src = states + (int64_t)(S - 1) * N * P + q;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (group_of<NB>(i) == G) sh.Vi[(S - 1) & 1][i][lane] = src[(int64_t)i * P];
  }
  if (S > 1) {
    const float* src = states + (int64_t)(S - 2) * N * P + q;
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (group_of<NB>(i) == G) pre[i] = src[(int64_t)i * P];
  }
  __syncthreads();
  for (int s = S - 1; s >= 0; --s) {
    const int b = s & 1;
    float Vb[N], A[N], T[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      Vb[i] = sh.Vb[b ^ 1][i][lane];
      A[i] = sh.Vi[b][i][lane];
    }
    SqGroup<NB, G>::adj(Vb, A, T);  // group G of 2 (Vb * V_in)
    const PairGeom geo = pair_geom(px, py, pz, sph[s]);
    {
      // This wave's share of the pair weights: W_lm = PAIR_lm hbar_lm on
      // its output group, 0 elsewhere (the pair adjoint is linear in W).
      float W[N], W0[NB];
#pragma unroll
      for (int l = 0; l < NB; ++l) {
#pragma unroll
        for (int m = -l; m <= l; ++m) {
          const int i = idx(l, m);
          const float w = group_of<NB>(i) == G ? SHV_PAIR[l][m < 0 ? -m : m] * (hbeta * T[i]) : 0.0f;
          W[i] = w;
          if (m == 0) W0[l] = w * SHV_ROW_0[l];
        }
      }
      float gvx, gvy, gvz, gr;
      pair_adjoint<NB>(geo, 1.0f, W, W0, gvx, gvy, gvz, gr);
      gpx -= gvx;
      gpy -= gvy;
      gpz -= gvz;
      const float4 tot = make_float4(wave_sum_last(gvx), wave_sum_last(gvy), wave_sum_last(gvz), wave_sum_last(gr));
      if (lane == 63) gs_row[s] = tot;
    }
    blocker_vec<NB>(geo, A);
    SqGroup<NB, G>::adj(Vb, A, T);  // group G of 2 (Vb * h)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (group_of<NB>(i) == G) sh.Vb[b][i][lane] = fmaf(hbeta, T[i], Vb[i]);
    if (s > 0) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (group_of<NB>(i) == G) sh.Vi[b ^ 1][i][lane] = pre[i];
    }
    if (s > 1) {
      const float* src = states + (int64_t)(s - 2) * N * P + q;
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (group_of<NB>(i) == G) pre[i] = src[(int64_t)i * P];
    }
    __syncthreads();
  }
  if (G > 0) {
    sh.gp[G - 1][0][lane] = gpx;
    sh.gp[G - 1][1][lane] = gpy;
    sh.gp[G - 1][2][lane] = gpz;
  }
  __syncthreads();
  if (G == 0 && ok && gpts) {
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      gpx += sh.gp[w][0][lane];
      gpy += sh.gp[w][1][lane];
      gpz += sh.gp[w][2][lane];
    }
    gpts[p] = gpx;
    gpts[P + p] = gpy;
    gpts[2 * P + p] = gpz;
  }
}

// gs_part: [4 * pair_blocks(P)][S], one row per (block, wave).
template <int NB>
__global__ __launch_bounds__(SHV_BLOCK, 2) void k_prod_bwd(const float* __restrict__ gvis,
                                                           const float* __restrict__ states,
                                                           const float* __restrict__ pts, int64_t P,
                                                           const float4* __restrict__ sph, int S, float hbeta,
                                                           float* __restrict__ gpts, float4* __restrict__ gs_part) {
  __shared__ ProdBwdShared<NB> sh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t bx = blockIdx.x;
  const int64_t p = bx * 64 + lane;
  const bool ok = p < P;
  switch (wave) {
    case 0: prod_bwd_group<NB, 0>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
    case 1: prod_bwd_group<NB, 1>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
    case 2: prod_bwd_group<NB, 2>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
    default: prod_bwd_group<NB, 3>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
  }
}

// ===========================================================================
// From 6 bands up: the product with a zonal function in its own frame.
//
// Rotated so that the sphere lies at +z, h is a function of z alone: at a
// latitude it multiplies every Fourier coefficient of V by one number.  One step
//   V <- V + beta R^-1 [ h (R V) ]
// rotates, takes the orders' Legendre transforms, multiplies, transforms back
// and rotates back: about 2,300 instructions per pair at 8 bands, against 10,800
// for the contraction with Gaunt coefficients and 4,750 for a general product
// through latitudes.  Only the increment goes through the rotations, so V keeps
// its own digits.  R = K^-1 Z(-theta) K Z(-phi) with Z the rotation about z
// (two products per entry) and K a quarter turn about x, 176 nonzero entries.
//
// The rotations are block-diagonal in the band l, the rest in the order m, so
// each of a block's four waves owns 16 of the 64 coefficients (8 bands) as
// whole bands and 16 as whole orders; the vector crosses LDS once each way per
// sphere, 16 values in and out per lane and two barriers, and V itself never
// leaves the registers of the waves that own its bands.
//
// Adjoint of a step: Vb <- Vb + beta (Vb * h) as forward, and with
// T1 = Vb * h, T2 = V_in * h, both in the sphere's frame,
//   dL/dt = beta int Vb V_in dh/dt, a sum over latitudes of the order-0 Fourier
//           coefficient of Vb V_in,
//   dL/ds = beta (< dR^-1 Vb, T2 > + < dR^-1 V_in, T1 >), because turning h one
//           way is turning both factors the other way: two bilinear forms per
//           band, the generators of the rotations about x and y.
// Neither Vb * V_in nor a pair adjoint over its coefficients is formed.  Each
// wave's share is linear and goes into its own row of the sphere partials.
//
// Bound by the chain's length: 1,252 waves at 20,000 receivers, 1.2 per SIMD.
// Measured there with 128 spheres at 8 bands: forward 905 -> 242 us, adjoint
// 1,870 -> 530 us.

template <int NB>
struct TurnTab;
#define SHV_TURNTAB(n)                                                                                  \
  template <>                                                                                           \
  struct TurnTab<n> {                                                                                   \
    static __device__ __forceinline__ constexpr int l_wave(int l) { return SHV_TURN_L_##n[l]; }         \
    static __device__ __forceinline__ constexpr int m_wave(int m) { return SHV_TURN_M_##n[m]; }         \
    static __device__ __forceinline__ constexpr float zonal(int t, int l) { return shv_zonal_rows_##n[t * n + l]; } \
  };
SHV_TURNTAB(6)
SHV_TURNTAB(7)
SHV_TURNTAB(8)
#undef SHV_TURNTAB

template <int L>
struct TurnBand;
#define SHV_TURNBAND(l)                                                                                         \
  template <>                                                                                                   \
  struct TurnBand<l> {                                                                                          \
    static __device__ __forceinline__ void turn(const float* v, float* o) { shv_turn_l##l(v, o); }              \
    static __device__ __forceinline__ void unturn(const float* v, float* o) { shv_unturn_l##l(v, o); }          \
    static __device__ __forceinline__ void torque(const float* v, const float* t, float& gx, float& gy) {       \
      shv_torque_l##l(v, t, gx, gy);                                                                            \
    }                                                                                                           \
  };
SHV_TURNBAND(0)
SHV_TURNBAND(1)
SHV_TURNBAND(2)
SHV_TURNBAND(3)
SHV_TURNBAND(4)
SHV_TURNBAND(5)
SHV_TURNBAND(6)
SHV_TURNBAND(7)
#undef SHV_TURNBAND

// f(integral constant l) for the bands of wave W.
template <int NB, int W, int L = 0, class F>
__device__ __forceinline__ void each_band(F f) {
  if constexpr (L < NB) {
    if constexpr (TurnTab<NB>::l_wave(L) == W) f(std::integral_constant<int, L>{});
    each_band<NB, W, L + 1>(f);
  }
}

// Cosine and sine of an angle, as its unit vector's coordinates brought to
// length 1 in FP32 (their m-th powers would carry an error of length m times).
__device__ __forceinline__ void unit_pair(float& c, float& s) {
  const float e = fmaf(-s, s, fmaf(-c, c, 1.0f));
  c = fmaf(c, 0.5f * e, c);
  s = fmaf(s, 0.5f * e, s);
}

// One pair's geometry in the sphere's frame: the angles' multiples, and the
// blocker (eps-free) at the latitudes, even and odd parts in z.
template <int NB>
struct TurnGeom {
  static constexpr int ROWS = LatTab<NB>::PAIRS + LatTab<NB>::EQ;
  PairGeom G;
  float cp[NB], sp[NB], ct[NB], st[NB];  // m phi, m theta
  float he[ROWS], ho[ROWS];              // h
  float de[ROWS], dq[ROWS];              // dh/dt / (2 pi) (adjoint only)
};

template <int NB, bool ADJ>
__device__ __forceinline__ void turn_geom(float px, float py, float pz, float4 q, TurnGeom<NB>& g) {
  g.G = pair_geom(px, py, pz, q);
  const float rho2 = fmaf(g.G.x, g.G.x, g.G.y * g.G.y);
  const bool pole = !(rho2 > 0.0f);  // the azimuth is free there
  const float ir = fast_rsqrt(pole ? 1.0f : rho2);
  float c = pole ? 1.0f : g.G.x * ir, s = pole ? 0.0f : g.G.y * ir;
  unit_pair(c, s);
  cs_powers<NB>(c, s, g.cp, g.sp);
  c = g.G.inv > 0.0f ? g.G.z : 1.0f;  // a sphere centred on the receiver has no direction (and h = 0)
  s = pole ? 0.0f : rho2 * ir;
  unit_pair(c, s);
  cs_powers<NB>(c, s, g.ct, g.st);
  float R[NB + 1], zg[NB];
  legendre_resid<NB>(g.G.t, g.G.u, R);
  cap_zonal<NB>(g.G.u, R, zg);
#pragma unroll
  for (int t = 0; t < TurnGeom<NB>::ROWS; ++t) {
    float h[2] = {0.0f, 0.0f}, d[2] = {0.0f, 0.0f};
#pragma unroll
    for (int l = 0; l < NB; ++l) {
      const float k = TurnTab<NB>::zonal(t, l);
      if (t >= LatTab<NB>::PAIRS && (l & 1)) continue;  // odd Legendre polynomials vanish at the equator
      h[l & 1] = l < 2 ? k * zg[l] : fmaf(k, zg[l], h[l & 1]);
      if constexpr (ADJ) d[l & 1] = l < 2 ? fmaf(-k, R[l], k) : fmaf(-k, R[l], d[l & 1] + k);
    }
    g.he[t] = h[0];
    g.ho[t] = h[1];
    g.de[t] = d[0];
    g.dq[t] = d[1];
  }
}

// Rotation of one band about z by the angle with multiples c, s (INV: by minus it).
template <int L, bool INV>
__device__ __forceinline__ void z_turn(float* v, const float* c, const float* s) {
#pragma unroll
  for (int m = 1; m <= L; ++m) {
    const float a = v[L + m], b = v[L - m], sm = INV ? -s[m] : s[m];
    v[L + m] = fmaf(c[m], a, -sm * b);
    v[L - m] = fmaf(sm, a, c[m] * b);
  }
}

// Band L of R f into the sphere's frame, and of R^-1 f out of it.
template <int NB, int L>
__device__ __forceinline__ void band_into(float* v, const TurnGeom<NB>& g) {
  float o[2 * L + 1];
  z_turn<L, true>(v, g.cp, g.sp);
  TurnBand<L>::turn(v, o);
  z_turn<L, true>(o, g.ct, g.st);
  TurnBand<L>::unturn(o, v);
}
template <int NB, int L>
__device__ __forceinline__ void band_out(float* v, const TurnGeom<NB>& g) {
  float o[2 * L + 1];
  TurnBand<L>::turn(v, o);
  z_turn<L, false>(o, g.ct, g.st);
  TurnBand<L>::unturn(o, v);
  z_turn<L, false>(v, g.cp, g.sp);
}

// One order's column (cosines SIN = false, sines true) times the zonal function:
// o_lm += the transposed transform of h times the transform of e.  With ADJ the
// same for a second vector x -> y, and gt += the two vectors' product at the
// latitudes times dh/dt.
template <int NB, bool SIN, bool ADJ>
__device__ __forceinline__ void zonal_column(int m, const float (&e)[NB * NB], const float (&x)[NB * NB],
                                             const TurnGeom<NB>& g, float (&o)[NB * NB], float (&y)[NB * NB],
                                             float& gt) {
  constexpr int PAIRS = LatTab<NB>::PAIRS, QP = Lat<NB>::QP;
#pragma unroll
  for (int t = 0; t < TurnGeom<NB>::ROWS; ++t) {
    const bool eq = t >= PAIRS;
    const float* __restrict__ Q = LatTab<NB>::rows() + t * QP;
    float a[2] = {0.0f, 0.0f}, b[2] = {0.0f, 0.0f};
#pragma unroll
    for (int l = m; l < NB; ++l) {
      const int s = (l - m) & 1;
      if (eq && s) continue;
      const int i = idx(l, SIN ? -m : m);
      const float k = Q[lat_at<NB>(m) + l - m];
      a[s] = l < m + 2 ? k * e[i] : fmaf(k, e[i], a[s]);
      if constexpr (ADJ) b[s] = l < m + 2 ? k * x[i] : fmaf(k, x[i], b[s]);
    }
    float ge, go, fe = 0.0f, fo = 0.0f;
    if (eq) {
      ge = g.he[t] * a[0];
      go = 0.0f;
      if constexpr (ADJ) {
        fe = g.he[t] * b[0];
        gt = fmaf(g.de[t] * a[0], b[0], gt);
      }
    } else {
      ge = fmaf(g.he[t], a[0], g.ho[t] * a[1]);
      go = fmaf(g.ho[t], a[0], g.he[t] * a[1]);
      if constexpr (ADJ) {
        fe = fmaf(g.he[t], b[0], g.ho[t] * b[1]);
        fo = fmaf(g.ho[t], b[0], g.he[t] * b[1]);
        gt = fmaf(g.de[t], fmaf(a[0], b[0], a[1] * b[1]), gt);
        gt = fmaf(g.dq[t], fmaf(a[0], b[1], a[1] * b[0]), gt);
      }
    }
#pragma unroll
    for (int l = m; l < NB; ++l) {
      const int s = (l - m) & 1;
      if (eq && s) continue;
      const int i = idx(l, SIN ? -m : m);
      const float k = Q[lat_at<NB>(m) + l - m];
      o[i] = t == 0 ? k * (s ? go : ge) : fmaf(k, s ? go : ge, o[i]);
      if constexpr (ADJ) y[i] = t == 0 ? k * (s ? fo : fe) : fmaf(k, s ? fo : fe, y[i]);
    }
  }
}

template <int NB>
struct TurnFwdShared {
  float A[NB * NB][64];  // R V
  float B[NB * NB][64];  // 2 h (R V)
};

template <int NB, int W>
__device__ __forceinline__ void turn_fwd_wave(TurnFwdShared<NB>& sh, int lane, int64_t p, bool ok,
                                              const float* __restrict__ pts, int64_t P,
                                              const float4* __restrict__ sph, int S, float hbeta,
                                              float* __restrict__ vis, float* __restrict__ states) {
  constexpr int N = NB * NB;
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  const float px = sel0(ok, pts[q]);
  const float py = sel0(ok, pts[P + q]);
  const float pz = sel0(ok, pts[2 * P + q]);
  float V[N];  // this wave's bands only
#pragma unroll
  for (int i = 0; i < N; ++i) V[i] = i == 0 ? 1.0f : 0.0f;
  for (int s = 0; s < S; ++s) {
    if (states && ok) {
      float* dst = states + (int64_t)s * N * P + p;
      each_band<NB, W>([&](auto l) {
#pragma unroll
        for (int i = l * l; i < (l + 1) * (l + 1); ++i) dst[(int64_t)i * P] = V[i];
      });
    }
    TurnGeom<NB> g;
    turn_geom<NB, false>(px, py, pz, sph[s], g);
    each_band<NB, W>([&](auto l) {
      float v[2 * l + 1];
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) v[i] = V[l * l + i];
      band_into<NB, l>(v, g);
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) sh.A[l * l + i][lane] = v[i];
    });
    __syncthreads();
    {
      float e[N], o[N], none;
#pragma unroll
      for (int m = 0; m < NB; ++m) {
        if (TurnTab<NB>::m_wave(m) != W) continue;
#pragma unroll
        for (int l = m; l < NB; ++l) {
          e[idx(l, m)] = sh.A[idx(l, m)][lane];
          e[idx(l, -m)] = sh.A[idx(l, -m)][lane];
        }
        zonal_column<NB, false, false>(m, e, e, g, o, o, none);
        if (m > 0) zonal_column<NB, true, false>(m, e, e, g, o, o, none);
#pragma unroll
        for (int l = m; l < NB; ++l) {
          sh.B[idx(l, m)][lane] = o[idx(l, m)];
          if (m > 0) sh.B[idx(l, -m)][lane] = o[idx(l, -m)];
        }
      }
    }
    __syncthreads();  // A is rewritten only after this, B only after the next one
    each_band<NB, W>([&](auto l) {
      float v[2 * l + 1];
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) v[i] = sh.B[l * l + i][lane];
      band_out<NB, l>(v, g);
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) V[l * l + i] = fmaf(hbeta, v[i], V[l * l + i]);
    });
  }
  if (vis && ok) {
    each_band<NB, W>([&](auto l) {
#pragma unroll
      for (int i = l * l; i < (l + 1) * (l + 1); ++i) vis[(int64_t)i * P + p] = V[i] * coef_inv<NB>(i);
    });
  }
}

template <int NB>
__global__ __launch_bounds__(SHV_BLOCK) void k_turn_fwd(const float* __restrict__ pts, int64_t P,
                                                        const float4* __restrict__ sph, int S, float hbeta,
                                                        float* __restrict__ vis, float* __restrict__ states) {
  __shared__ TurnFwdShared<NB> sh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t p = (int64_t)blockIdx.x * 64 + lane;
  const bool ok = p < P;
  switch (wave) {
    case 0: turn_fwd_wave<NB, 0>(sh, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
    case 1: turn_fwd_wave<NB, 1>(sh, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
    case 2: turn_fwd_wave<NB, 2>(sh, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
    default: turn_fwd_wave<NB, 3>(sh, lane, p, ok, pts, P, sph, S, hbeta, vis, states); break;
  }
}

template <int NB>
struct TurnBwdShared {
  float A[2][NB * NB][64];  // R V_in, R Vb
  float B[2][NB * NB][64];  // 2 h (R V_in), 2 h (R Vb)
  float gp[3][3][64];       // receiver-gradient partials of waves 1..3
};

template <int NB, int W>
__device__ __forceinline__ void turn_bwd_wave(TurnBwdShared<NB>& sh, int lane, int64_t bx, int64_t p, bool ok,
                                              const float* __restrict__ gvis, const float* __restrict__ states,
                                              const float* __restrict__ pts, int64_t P,
                                              const float4* __restrict__ sph, int S, float hbeta,
                                              float* __restrict__ gpts, float4* __restrict__ gs_part) {
  constexpr int N = NB * NB;
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  const float px = sel0(ok, pts[q]);
  const float py = sel0(ok, pts[P + q]);
  const float pz = sel0(ok, pts[2 * P + q]);
  float gpx = 0.0f, gpy = 0.0f, gpz = 0.0f;
  float4* gs_row = gs_part + (bx * 4 + W) * S;
  // This wave's bands of the cotangent (zero on tail lanes, so they add nothing
  // to the sphere sums) and of each step's input, loaded one sphere ahead.
  float Vb[N], V[N];
  each_band<NB, W>([&](auto l) {
#pragma unroll
    for (int i = l * l; i < (l + 1) * (l + 1); ++i) Vb[i] = sel0(ok, gvis[(int64_t)i * P + q]) * cot_scale<NB>(i);
  });
  const auto load_state = [&](int s) {
    const float* src = states + (int64_t)s * N * P + q;
    each_band<NB, W>([&](auto l) {
#pragma unroll
      for (int i = l * l; i < (l + 1) * (l + 1); ++i) V[i] = src[(int64_t)i * P];
    });
  };
  if (S > 0) load_state(S - 1);
  for (int s = S - 1; s >= 0; --s) {
    TurnGeom<NB> g;
    turn_geom<NB, true>(px, py, pz, sph[s], g);
    each_band<NB, W>([&](auto l) {
      constexpr int b = l * l;
      float v[2 * l + 1], w[2 * l + 1];
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) {
        v[i] = V[b + i];
        w[i] = Vb[b + i];
      }
      band_into<NB, l>(v, g);
      band_into<NB, l>(w, g);
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) {
        sh.A[0][b + i][lane] = v[i];
        sh.A[1][b + i][lane] = w[i];
      }
    });
    __syncthreads();
    float gt = 0.0f;
    {
      float e[N], x[N], o[N], y[N];
#pragma unroll
      for (int m = 0; m < NB; ++m) {
        if (TurnTab<NB>::m_wave(m) != W) continue;
#pragma unroll
        for (int l = m; l < NB; ++l) {
          e[idx(l, m)] = sh.A[0][idx(l, m)][lane];
          x[idx(l, m)] = sh.A[1][idx(l, m)][lane];
          e[idx(l, -m)] = sh.A[0][idx(l, -m)][lane];
          x[idx(l, -m)] = sh.A[1][idx(l, -m)][lane];
        }
        float gm = 0.0f;
        zonal_column<NB, false, true>(m, e, x, g, o, y, gm);
        if (m > 0) zonal_column<NB, true, true>(m, e, x, g, o, y, gm);
        gt = m > 0 ? fmaf(2.0f, gm, gt) : gt + gm;
#pragma unroll
        for (int l = m; l < NB; ++l) {
          sh.B[0][idx(l, m)][lane] = o[idx(l, m)];
          sh.B[1][idx(l, m)][lane] = y[idx(l, m)];
          if (m > 0) {
            sh.B[0][idx(l, -m)][lane] = o[idx(l, -m)];
            sh.B[1][idx(l, -m)][lane] = y[idx(l, -m)];
          }
        }
      }
    }
    __syncthreads();  // A is rewritten only after this, B only after the next one
    float tx = 0.0f, ty = 0.0f;
    each_band<NB, W>([&](auto l) {
      constexpr int b = l * l;
      float t[2 * l + 1], v[2 * l + 1];
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) {
        t[i] = sh.B[0][b + i][lane];   // 2 V_in * h
        v[i] = sh.A[1][b + i][lane];   // R Vb, this wave's own
      }
      TurnBand<l>::torque(v, t, tx, ty);
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) {
        t[i] = sh.B[1][b + i][lane];   // 2 Vb * h
        v[i] = sh.A[0][b + i][lane];   // R V_in
      }
      TurnBand<l>::torque(v, t, tx, ty);
      band_out<NB, l>(t, g);
#pragma unroll
      for (int i = 0; i < 2 * l + 1; ++i) Vb[b + i] = fmaf(hbeta, t[i], Vb[b + i]);
    });
    if (s > 0) load_state(s - 1);
    // Chain rule in the frame's tangent directions: along theta (R^-1 x) and
    // along phi (R^-1 y), then through s = v / |v| and t(|v|, r).
    const float f = hbeta * SHV_SQRT_4PI;
    tx *= f * g.G.inv;
    ty *= f * g.G.inv;
    const float Gt = gt * (f * SHV_TWO_PI);
    const float cp = g.cp[1], sp = g.sp[1], ct = g.ct[1], st = g.st[1];
    float gvx = fmaf(tx, ct * cp, -ty * sp);
    float gvy = fmaf(tx, ct * sp, ty * cp);
    float gvz = -tx * st;
    float gr = 0.0f;
    if (g.G.t > 0.0f) {
      const float k = Gt * g.G.rs * fast_rcp(g.G.t) * g.G.inv;  // dLoss/dt * (-dt/dr); t > 0 here
      const float kd = k * g.G.rs;                              // dLoss/dt * dt/d|v|
      gvx = fmaf(kd, g.G.x, gvx);
      gvy = fmaf(kd, g.G.y, gvy);
      gvz = fmaf(kd, g.G.z, gvz);
      gr = -k;
    }
    gpx -= gvx;
    gpy -= gvy;
    gpz -= gvz;
    const float tot = wave_sum4(gvx, gvy, gvz, gr);
    if ((lane & 15) == 15) reinterpret_cast<float*>(gs_row + s)[lane >> 4] = tot;
  }
  if (W > 0) {
    sh.gp[W - 1][0][lane] = gpx;
    sh.gp[W - 1][1][lane] = gpy;
    sh.gp[W - 1][2][lane] = gpz;
  }
  __syncthreads();
  if (W == 0 && ok && gpts) {
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      gpx += sh.gp[w][0][lane];
      gpy += sh.gp[w][1][lane];
      gpz += sh.gp[w][2][lane];
    }
    gpts[p] = gpx;
    gpts[P + p] = gpy;
    gpts[2 * P + p] = gpz;
  }
}

// gs_part: [4 * pair_blocks(P)][S], one row per (block, wave).
template <int NB>
__global__ __launch_bounds__(SHV_BLOCK, 2) void k_turn_bwd(const float* __restrict__ gvis,
                                                           const float* __restrict__ states,
                                                           const float* __restrict__ pts, int64_t P,
                                                           const float4* __restrict__ sph, int S, float hbeta,
                                                           float* __restrict__ gpts, float4* __restrict__ gs_part) {
  __shared__ TurnBwdShared<NB> sh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t bx = blockIdx.x;
  const int64_t p = bx * 64 + lane;
  const bool ok = p < P;
  switch (wave) {
    case 0: turn_bwd_wave<NB, 0>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
    case 1: turn_bwd_wave<NB, 1>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
    case 2: turn_bwd_wave<NB, 2>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
    default: turn_bwd_wave<NB, 3>(sh, lane, bx, p, ok, gvis, states, pts, P, sph, S, hbeta, gpts, gs_part); break;
  }
}

// ---------------------------------------------------------------------------
// Launchers for one band count (instantiated per band count in shv_nb.hip).
// beta = 1 - e^-eps is formed in double precision and rounded once.

inline float prod_half_beta(float eps) { return (float)(-0.5 * std::expm1(-(double)eps)); }

template <int NB>
hipError_t prod_fwd_nb(const float* pts, int64_t P, const float* sph, int S, float eps, float* vis, float* states,
                       hipStream_t st) {
  if constexpr (Lat<NB>::USE) {
    k_turn_fwd<NB><<<(unsigned)pair_blocks(P), SHV_BLOCK, 0, st>>>(pts, P, (const float4*)sph, S,
                                                                   prod_half_beta(eps), vis, states);
  } else {
    k_prod_fwd<NB><<<(unsigned)pair_blocks(P), SHV_BLOCK, 0, st>>>(pts, P, (const float4*)sph, S,
                                                                   prod_half_beta(eps), vis, states);
  }
  return hipGetLastError();
}

template <int NB>
hipError_t prod_bwd_nb(const float* gvis, const float* states, const float* pts, int64_t P, const float* sph, int S,
                       float eps, float* gpts, float* gs_part, hipStream_t st) {
  if constexpr (Lat<NB>::USE) {
    k_turn_bwd<NB><<<(unsigned)pair_blocks(P), SHV_BLOCK, 0, st>>>(gvis, states, pts, P, (const float4*)sph, S,
                                                                   prod_half_beta(eps), gpts, (float4*)gs_part);
  } else {
    k_prod_bwd<NB><<<(unsigned)pair_blocks(P), SHV_BLOCK, 0, st>>>(gvis, states, pts, P, (const float4*)sph, S,
                                                                   prod_half_beta(eps), gpts, (float4*)gs_part);
  }
  return hipGetLastError();
}

}  // namespace shv
