// Truncated products of SH vectors through latitudes, from 6 bands up.
//
// A product a * b of two n-band functions, projected back on n bands, is exact
// on a product grid.  At a latitude z each function is a trigonometric
// polynomial of degree n - 1 in the azimuth, found by a Legendre transform per
// order m; the product of the two is the convolution of their Fourier
// coefficients; the projection is the transposed transform, summed over the
// Gauss-Legendre latitudes of degree 3 n - 3 (11 at 8 bands).  The latitudes
// go in pairs +-z, whose transforms share their even and odd parts in l - m.
// At 8 bands a square takes about 2,750 multiply-adds and a product of two
// vectors 4,750, against 8,700 and 10,800 for the sparse contraction with the
// 12,868 Gaunt coefficients; at 6 bands 1,210 and 2,020 against 2,200 and
// 2,870; at 5 bands the two meet, and the contraction stays.
//
// A product's outputs split by order: the coefficients of one order |m| need
// one order of the Fourier product, and all of the factors' transforms.  A
// four-wave kernel gives each wave a group of whole orders (about 1,070 and
// 1,950 instructions), every wave repeating the transforms.  Every output is
// the same chain of operations in the same order whichever group asks for it,
// so the one-wave and four-wave kernels agree bit for bit.  The rows are
// unrolled with their constants as literals: a rolled loop with scalar loads of
// the constants waits for them at every row (four-wave forward and adjoint of
// 20,000 receivers 24.0 and 40.5 us rolled, 21.1 and 36.6 us unrolled; with the
// next row's constants loaded ahead 26.4 and 43.0 us, the scalar moves costing
// more than the wait).
//
// Measured (fused kernels at 8 bands, 4 squarings, contraction -> latitudes):
// 20,000 receivers 30.5 -> 21.1 us forward, 43.3 -> 36.6 us adjoint; 262,144
// receivers 196 -> 128 and 356 -> 313 us.  What bounds them now: the adjoint's
// set-up (shading adjoint, lighting tile) and, with one or two waves per SIMD,
// the 5.4 cycles between the instructions of one wave.
//
// Coefficients inside a product are scaled: e_l0 = E_l0 / sqrt(4 pi) and
// e_lm = E_lm / sqrt(8 pi).  The function's Fourier coefficient of order
// m >= 0 is then A_m - i B_m with A_m = sum_l Q_lm e_lm, B_m = sum_l Q_lm e_l-m,
// one table Q serving the transform and its transpose, and e_00 is the mean.
// The mean of one factor is multiplied exactly and kept out of the transform,
// (e_00 + d) b = e_00 b + d b, which about halves the rounding error of the
// exponential against the contraction with Gaunt coefficients.  Cotangents
// h are carried as sqrt(4 pi) times that scale, so that the same product serves.
#pragma once

#include "shv_device.h"

namespace shv {

template <int NB>
struct LatTab {
  static constexpr int PAIRS = 0, EQ = 0;
};
#define SHV_LATTAB(n)                                                                             \
  template <>                                                                                     \
  struct LatTab<n> {                                                                              \
    static constexpr int PAIRS = SHV_LAT_PAIRS_##n, EQ = SHV_LAT_EQ_##n;                          \
    static __device__ __forceinline__ const float* rows() { return shv_lat_rows_##n; }            \
  };
SHV_LATTAB(6)
SHV_LATTAB(7)
SHV_LATTAB(8)
#undef SHV_LATTAB

template <int NB>
struct Lat {
  static constexpr bool USE = LatTab<NB>::PAIRS > 0;
  static constexpr int QP = (NB * (NB + 1) / 2 + 3) / 4 * 4;  // padded entries of a row
};

// 1 / scale, the scale, and the scale times sqrt(4 pi) of coefficient i (1 for
// band counts that don't scale).
__device__ __forceinline__ constexpr int lat_zonal(int i) {
  int l = 0;
  while ((l + 1) * (l + 1) <= i) ++l;
  return i == l * l + l;
}
template <int NB>
__device__ __forceinline__ constexpr float coef_inv(int i) {
  return Lat<NB>::USE ? SHV_LAT_INV[lat_zonal(i) ? 0 : 1] : 1.0f;
}
template <int NB>
__device__ __forceinline__ constexpr float coef_scale(int i) {
  return Lat<NB>::USE ? SHV_LAT_SCALE[lat_zonal(i) ? 0 : 1] : 1.0f;
}
template <int NB>
__device__ __forceinline__ constexpr float cot_scale(int i) {
  return Lat<NB>::USE && !lat_zonal(i) ? 0.70710678118654752f : 1.0f;
}
// The constant function 1.
template <int NB>
__device__ __forceinline__ constexpr float one_coef() { return Lat<NB>::USE ? 1.0f : SHV_SQRT_4PI; }

template <int NB>
__device__ __forceinline__ constexpr int group_of(int i);

// Whether group G (-1: all) holds the outputs of order m.
template <int NB, int G>
__device__ __forceinline__ constexpr bool lat_has(int m) { return G < 0 || group_of<NB>(idx(m, m)) == G; }

// First entry of order m in a row (l = m .. NB - 1 follow).
template <int NB>
__device__ __forceinline__ constexpr int lat_at(int m) { return m * NB - m * (m - 1) / 2; }

// Order m of the Fourier coefficients of the function with coefficients e(i), at
// z (index 0) and -z (1), or at the equator (EQ; the odd terms vanish); without
// its mean unless MEAN.
template <int NB, bool EQ, bool MEAN, class Coef>
__device__ __forceinline__ void lat_up_order(Coef e, const float* __restrict__ Q, int m, float (&A)[2][NB],
                                             float (&B)[2][NB]) {
#pragma clang fp contract(off)  // the sums of two products below round alike in every kernel
  float a[2] = {0.0f, 0.0f}, b[2] = {0.0f, 0.0f};
  bool on[2] = {false, false};
#pragma unroll
  for (int l = m; l < NB; ++l) {
    const int s = (l - m) & 1;
    if ((l == 0 && !MEAN) || (EQ && s)) continue;
    const float t = Q[lat_at<NB>(m) + l - m];
    a[s] = on[s] ? fmaf(t, e(idx(l, m)), a[s]) : t * e(idx(l, m));
    if (m > 0) b[s] = on[s] ? fmaf(t, e(idx(l, -m)), b[s]) : t * e(idx(l, -m));
    on[s] = true;
  }
  A[0][m] = EQ ? a[0] : a[0] + a[1];
  A[1][m] = EQ ? 0.0f : a[0] - a[1];
  B[0][m] = EQ ? b[0] : b[0] + b[1];
  B[1][m] = EQ ? 0.0f : b[0] - b[1];
}

template <int NB, bool EQ, bool MEAN, class Coef>
__device__ __forceinline__ void lat_up(Coef e, const float* __restrict__ Q, float (&A)[2][NB], float (&B)[2][NB]) {
#pragma unroll
  for (int m = 0; m < NB; ++m) lat_up_order<NB, EQ, MEAN>(e, Q, m, A, B);
}

// Order m of half the square of c = A - i B (the weight's factor 2 makes it whole).
template <int NB>
__device__ __forceinline__ void lat_square(const float (&A)[NB], const float (&B)[NB], int m, float& da, float& db) {
  if (m == 0) {
    da = (0.5f * A[0]) * A[0];
#pragma unroll
    for (int t = 1; t < NB; ++t) da = fmaf(B[t], B[t], fmaf(A[t], A[t], da));
    db = 0.0f;
    return;
  }
  da = A[0] * A[m];
  db = A[0] * B[m];
#pragma unroll
  for (int t = 1; 2 * t <= m; ++t) {  // c_t c_(m-t)
    if (2 * t < m) {
      da = fmaf(-B[t], B[m - t], fmaf(A[t], A[m - t], da));
      db = fmaf(B[t], A[m - t], fmaf(A[t], B[m - t], db));
    } else {
      da = fmaf(-0.5f * B[t], B[t], fmaf(0.5f * A[t], A[t], da));
      db = fmaf(A[t], B[t], db);
    }
  }
#pragma unroll
  for (int t = 1; m + t < NB; ++t) {  // conj(c_t) c_(m+t)
    da = fmaf(B[t], B[m + t], fmaf(A[t], A[m + t], da));
    db = fmaf(-B[t], A[m + t], fmaf(A[t], B[m + t], db));
  }
}

// Order m of the product of A - i B and X - i Y.
template <int NB>
__device__ __forceinline__ void lat_mul(const float (&A)[NB], const float (&B)[NB], const float (&X)[NB],
                                        const float (&Y)[NB], int m, float& da, float& db) {
  if (m == 0) {
    float s = A[1] * X[1];
    s = fmaf(B[1], Y[1], s);
#pragma unroll
    for (int t = 2; t < NB; ++t) s = fmaf(B[t], Y[t], fmaf(A[t], X[t], s));
    da = fmaf(2.0f, s, A[0] * X[0]);
    db = 0.0f;
    return;
  }
  da = fmaf(A[0], X[m], A[m] * X[0]);
  db = fmaf(A[0], Y[m], B[m] * X[0]);
#pragma unroll
  for (int t = 1; t < m; ++t) {
    da = fmaf(-B[t], Y[m - t], fmaf(A[t], X[m - t], da));
    db = fmaf(B[t], X[m - t], fmaf(A[t], Y[m - t], db));
  }
#pragma unroll
  for (int t = 1; m + t < NB; ++t) {
    da = fmaf(B[t], Y[m + t], fmaf(A[t], X[m + t], da));
    da = fmaf(B[m + t], Y[t], fmaf(A[m + t], X[t], da));
    db = fmaf(-B[t], X[m + t], fmaf(A[t], Y[m + t], db));
    db = fmaf(-A[m + t], Y[t], fmaf(B[m + t], X[t], db));
  }
}

// One row of a product from the factors' Fourier coefficients: o += its share
// (o = its share for the first row), for the orders of group G.  SQUARE: (e -
// mean)^2, else twice (e - mean) h.
template <int NB, int G, bool SQUARE, bool EQ>
__device__ __forceinline__ void lat_down(const float (&A)[2][NB], const float (&B)[2][NB], const float (&X)[2][NB],
                                         const float (&Y)[2][NB], const float* __restrict__ Q, bool first,
                                         float (&o)[NB * NB]) {
#pragma unroll
  for (int m = 0; m < NB; ++m) {
    if (!lat_has<NB, G>(m)) continue;
    float da[2] = {0.0f, 0.0f}, db[2] = {0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < (EQ ? 1 : 2); ++s) {
      if constexpr (SQUARE) lat_square<NB>(A[s], B[s], m, da[s], db[s]);
      else lat_mul<NB>(A[s], B[s], X[s], Y[s], m, da[s], db[s]);
    }
    const float ea = EQ ? da[0] : da[0] + da[1], oa = da[0] - da[1];
    const float eb = EQ ? db[0] : db[0] + db[1], ob = db[0] - db[1];
#pragma unroll
    for (int l = m; l < NB; ++l) {
      const bool odd = ((l - m) & 1) != 0;
      if (EQ && odd) continue;
      const float t = Q[lat_at<NB>(m) + l - m];
      const float va = odd ? oa : ea, vb = odd ? ob : eb;
      o[idx(l, m)] = first ? t * va : fmaf(t, va, o[idx(l, m)]);
      if (m > 0) o[idx(l, -m)] = first ? t * vb : fmaf(t, vb, o[idx(l, -m)]);
    }
  }
}

template <int NB, int G, bool SQUARE, bool EQ, class Coef>
__device__ __forceinline__ void lat_row(Coef e, const float (&h)[NB * NB], const float* __restrict__ Q, bool first,
                                        float (&o)[NB * NB]) {
  float A[2][NB], B[2][NB], X[2][NB], Y[2][NB];
  lat_up<NB, EQ, false>(e, Q, A, B);
  if constexpr (!SQUARE) lat_up<NB, EQ, true>([&](int i) { return h[i]; }, Q, X, Y);
  lat_down<NB, G, SQUARE, EQ>(A, B, X, Y, Q, first, o);
}

// The outputs of group G (-1: all): o = e * e (SQUARE) or o = 2 (h * e), e(i)
// the coefficients of e.  between() is called before each row.
template <int NB, int G, bool SQUARE, class Coef, class Between>
__device__ __forceinline__ void lat_product(Coef e, const float (&h)[NB * NB], float (&o)[NB * NB], Between between) {
  constexpr int N = NB * NB, QP = Lat<NB>::QP;
  const float* __restrict__ Q = LatTab<NB>::rows();
#pragma unroll
  for (int t = 0; t < LatTab<NB>::PAIRS; ++t) {
    between();
    lat_row<NB, G, SQUARE, false>(e, h, Q + t * QP, t == 0, o);
  }
  if constexpr (LatTab<NB>::EQ > 0) {
    between();
    lat_row<NB, G, SQUARE, true>(e, h, Q + LatTab<NB>::PAIRS * QP, false, o);
  }
  const float t0 = 2.0f * e(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (G >= 0 && group_of<NB>(i) != G) continue;
    if constexpr (SQUARE) o[i] = i == 0 ? fmaf(e(0), e(0), o[0]) : fmaf(t0, e(i), o[i]);
    else o[i] = fmaf(t0, h[i], o[i]);
  }
}

template <int NB, int G, bool SQUARE>
__device__ __forceinline__ void lat_product(const float (&e)[NB * NB], const float (&h)[NB * NB],
                                            float (&o)[NB * NB]) {
  lat_product<NB, G, SQUARE>([&](int i) { return e[i]; }, h, o, [] {});
}

// The same product by the four waves of a block, wave G holding the
// coefficients of its own orders only, of the factors and of the outputs: it
// transforms its orders up, the waves exchange Fourier coefficients through LDS
// (lane by lane, 16 bytes per order, row and factor), and each forms its own
// outputs from all of them.  Against exchanging coefficients and transforming
// all of them in every wave, the transforms up, half of a wave's work in the
// adjoint and a third in the squaring, are done once.  PH: phases of rows, which
// bound the buffer.  PIN: the sums are formed before each phase's last barrier;
// where a branch follows, the compiler otherwise moves them behind it and holds
// all that was read.  The bits are those of lat_product.  Ends with a barrier.
// Bound: up to a few blocks per CU by what one wave issues (an instruction in
// four cycles at best) and by the barriers; forward and adjoint of the
// exponential, k = 4, us before and after: 6 bands 20.0 + 38.8 -> 18.3 + 36.2 at
// 50,000 receivers, 8 bands 40.0 + 77.4 -> 37.5 + 74.4 at 65,000, 20.9 + 36.1 ->
// 21.1 + 36.5 at 20,000.
template <int NB, bool SQUARE, int PH>
struct LatShared {
  static constexpr int ROWS = (LatTab<NB>::PAIRS + LatTab<NB>::EQ + PH - 1) / PH, F = SQUARE ? 1 : 2;
  float4 q[ROWS * F * NB][64];
  float mean[64];
};

template <int NB, int G, bool SQUARE, int PH, bool PIN = false>
__device__ __forceinline__ void lat_product4(const float (&e)[NB * NB], const float (&h)[NB * NB], float (&o)[NB * NB],
                                             LatShared<NB, SQUARE, PH>& sh, int lane) {
  constexpr int N = NB * NB, QP = Lat<NB>::QP, PAIRS = LatTab<NB>::PAIRS, ROWS = PAIRS + LatTab<NB>::EQ;
  constexpr int PER = LatShared<NB, SQUARE, PH>::ROWS, F = LatShared<NB, SQUARE, PH>::F;
  const float* __restrict__ Q = LatTab<NB>::rows();
  const auto ce = [&](int i) { return e[i]; };
  const auto ch = [&](int i) { return h[i]; };
  if (lat_has<NB, G>(0)) sh.mean[lane] = e[0];
  float t0 = 0.0f;
#pragma unroll
  for (int ph = 0; ph < PH; ++ph) {
    float A[PER][2][NB], B[PER][2][NB], X[PER][2][NB], Y[PER][2][NB];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int t = ph * PER + u;
      if (t >= ROWS) continue;
#pragma unroll
      for (int m = 0; m < NB; ++m) {
        if (!lat_has<NB, G>(m)) continue;
        if (t < PAIRS) lat_up_order<NB, false, false>(ce, Q + t * QP, m, A[u], B[u]);
        else lat_up_order<NB, true, false>(ce, Q + t * QP, m, A[u], B[u]);
        sh.q[(u * F) * NB + m][lane] = make_float4(A[u][0][m], A[u][1][m], B[u][0][m], B[u][1][m]);
        if constexpr (!SQUARE) {
          if (t < PAIRS) lat_up_order<NB, false, true>(ch, Q + t * QP, m, X[u], Y[u]);
          else lat_up_order<NB, true, true>(ch, Q + t * QP, m, X[u], Y[u]);
          sh.q[(u * F + 1) * NB + m][lane] = make_float4(X[u][0][m], X[u][1][m], Y[u][0][m], Y[u][1][m]);
        }
      }
    }
    __syncthreads();
    if (ph == 0) t0 = 2.0f * sh.mean[lane];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int t = ph * PER + u;
      if (t >= ROWS) continue;
#pragma unroll
      for (int m = 0; m < NB; ++m) {
        if (lat_has<NB, G>(m)) continue;
        const float4 v = sh.q[(u * F) * NB + m][lane];
        A[u][0][m] = v.x;
        A[u][1][m] = v.y;
        B[u][0][m] = v.z;
        B[u][1][m] = v.w;
        if constexpr (!SQUARE) {
          const float4 w = sh.q[(u * F + 1) * NB + m][lane];
          X[u][0][m] = w.x;
          X[u][1][m] = w.y;
          Y[u][0][m] = w.z;
          Y[u][1][m] = w.w;
        }
      }
      if (t < PAIRS) lat_down<NB, G, SQUARE, false>(A[u], B[u], X[u], Y[u], Q + t * QP, t == 0, o);
      else lat_down<NB, G, SQUARE, true>(A[u], B[u], X[u], Y[u], Q + t * QP, t == 0, o);
    }
    if constexpr (PIN) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (group_of<NB>(i) == G) asm volatile("" : "+v"(o[i]));
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (group_of<NB>(i) != G) continue;
    if constexpr (SQUARE) o[i] = i == 0 ? fmaf(e[0], e[0], o[0]) : fmaf(t0, e[i], o[i]);
    else o[i] = fmaf(t0, h[i], o[i]);
  }
}

}  // namespace shv
