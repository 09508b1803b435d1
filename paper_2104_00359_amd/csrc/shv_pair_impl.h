// Pair kernels: the O(P * S) part of the method (Sec. 3.3.2).
//
// Forward, per (receiver x, sphere i): direction s = (c - x)/|c - x|, cap
// half-angle alpha = asin(r/|c - x|), t = cos(alpha); the log-blocker
// -eps * 1[w . s >= t] (Eq. 13) has zonal coefficients g_l(t) about s, and
// rotating them to s multiplies by y_lm(s).  The kernel accumulates
//   F'_lm(x) = sum_i a_l(t_i) rho_l^|m|(s_z) T_m(s_x, s_y)
// in registers, a_l and rho_l^m being the g_l and r_l^m of the basis whose
// constants are left out (shv_device.h); the factor eps * PAIR[l][|m|] that
// turns F' into the log-visibility F is applied once per receiver by the
// exponential kernel.
//
// Backward: per pair the terms are recomputed (nothing per pair is stored).
// With W_lm = dLoss/dF'_lm:
//   dLoss/dt  = -sum_lm W_lm (l + 1) p_l(t) rho_l^|m| T_m   (p_l: monic P_l)
//   dLoss/ds  = grad of sum_lm W_lm a_l rho_l^|m| T_m, projected on the tangent
//   plane, then chained through s = v/|v|, t = sqrt(1 - r^2/|v|^2), v = c - x.
// Receiver gradients stay in registers; a sphere's four gradient values are
// summed over the wave together (a transposed reduction: DPP moves and
// gfx950's permlane swaps, no LDS), written per sphere to LDS by the wave
// that owns the sphere, and stored as per-block partials reduced by a second
// deterministic pass.
//
// Layout: one receiver per lane.  A block holds 64 receivers and 4 waves;
// grid.y splits the sphere set into chunks and the block's chunk is split
// again over its 4 waves (sphere w, w + 4, ...), so small receiver sets still
// fill 256 CUs.  The waves' partial sums are combined through LDS in wave
// order.  The block's chunk of sphere records is staged in LDS once and read
// back as wave-uniform broadcasts (measured faster than scalar loads of each
// record: pair adjoint 748 -> 703 us at 8 bands on the 64-scene batch).
//
// Bound: FP32 issue, and in launches of 100 us and more the clock that the card
// holds under it (2.05 GHz of 2.4).  At 8 bands a pair takes 172 instructions
// forward and 390 backward, its sums over the wave included (206 and 443 with
// recurrences along l and the Bonnet recurrence of the cap).  Multiply-adds
// with a scalar operand, selects, compares, minima and maxima issue at half
// rate and reciprocals and roots at a quarter, so the loops hold constants as
// literals, clamp by modifier, and form 1 - t without a division.  The 64-scene
// batch, before and after, us, the fastest of twenty launches: forward 276 -> 222
// at 8 bands, 279 -> 219 at 6, 149 -> 115 at 4; adjoint 627 -> 485, 620 -> 490,
// 343 -> 262.

#pragma once

#include "shv_batch.h"
#include "shv_launch.h"
#include "shv_shade_common.h"

namespace shv {

struct PairGeom {
  float x, y, z;  // unit direction receiver -> centre
  float inv;      // 1 / |c - x| (0 for a sphere centred on the receiver)
  float rs;       // r / |c - x|
  float s2, t2;   // sin^2 and cos^2 of alpha: rs^2 and 1 - rs^2; 1 and 0 when the receiver is inside the sphere
  float t;        // cos(alpha)
  float u;        // 1 - t
};

__device__ __forceinline__ PairGeom pair_geom(float px, float py, float pz, float4 q) {
  PairGeom g;
  const float vx = q.x - px, vy = q.y - py, vz = q.z - pz;
  const float d2 = fmaf(vx, vx, fmaf(vy, vy, vz * vz));
  g.inv = d2 > 0.0f ? fast_rsqrt(d2) : 0.0f;
  g.x = vx * g.inv;
  g.y = vy * g.inv;
  g.z = vz * g.inv;
  g.rs = q.w * g.inv;
  g.s2 = fminf(g.rs * g.rs, 1.0f);
  g.t2 = __builtin_amdgcn_fmed3f(fmaf(-g.rs, g.rs, 1.0f), 0.0f, 1.0f);
  g.t = fast_sqrt(g.t2);
  // u solves u^2 - 2 u + s2 = 0; from u = 1 - t, whose error is one of t, the
  // step leaves u times that error: small caps keep their digits.
  const float u = 1.0f - g.t;
  g.u = 0.5f * fmaf(u, u, g.s2);  // = 1 when inside (t = 0)
  return g;
}

// The sphere chunk is needed during the sphere loop, X only after it: they
// share the storage (a barrier separates them), so staging the spheres costs
// the forward no LDS at 4 or more bands.  The waves' partial sums are
// exchanged half of the coefficients at a time, which halves X and lets more
// blocks share a CU.
template <int NB>
struct PairFwdHalf {
  static constexpr int N = NB * NB;
  static constexpr int H = (N + 1) / 2;  // coefficients per exchange
};
template <int NB>
union PairFwdShared {
  float X[SHV_WAVES_PER_BLOCK][PairFwdHalf<NB>::H][64];
  float4 sph[SHV_MAX_CHUNK];
};

// One block of the pair forward: receivers [64 bx, 64 bx + 64), sphere chunk
// by.  Blocks of chunk 0 also build M(L), block m_idx of m_count taking every
// m_count-th entry.
template <int NB>
__device__ __forceinline__ void pair_fwd_item(const float* __restrict__ pts, int64_t P, const float4* __restrict__ sph,
                                              int S, int chunk, float* __restrict__ Fpart,
                                              const float* __restrict__ L, float* __restrict__ M, int64_t bx, int by,
                                              int64_t m_idx, int64_t m_count, PairFwdShared<NB>& sh) {
  constexpr int N = NB * NB;
  auto& X = sh.X;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t p = bx * 64 + lane;
  const bool ok = p < P;
  const int s0 = by * chunk;
  const int s1 = min(S, s0 + chunk);
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  const float px = sel0(ok, pts[q]);
  const float py = sel0(ok, pts[P + q]);
  const float pz = sel0(ok, pts[2 * P + q]);

  float acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = 0.0f;
  // The DC coefficient sets V's overall scale through exp(F_0 / sqrt(4 pi)),
  // so its sum over spheres is compensated (Kahan).
  float dc_comp = 0.0f;

  for (int j = threadIdx.x; j < s1 - s0; j += SHV_BLOCK) sh.sph[j] = sph[s0 + j];
  __syncthreads();
  const float one = vector_one();
  for (int s = s0 + wave; s < s1; s += SHV_WAVES_PER_BLOCK) {
    const PairGeom G = pair_geom(px, py, pz, sh.sph[s - s0]);
    float g[NB], C[NB], Sn[NB], r[2][NB];
    cap_terms<NB>(G.t, G.u, G.s2, g);
    cs_powers<NB>(G.x, G.y, C, Sn);
    legendre_monic<NB>(G.z, r[0]);
    {
      const float y = g[0] - dc_comp;
      const float t = acc[0] + y;
      dc_comp = (t - acc[0]) - y;
      acc[0] = t;
    }
#pragma unroll
    for (int l = 1; l < NB; ++l) acc[idx(l, 0)] = fmaf(g[l], r[0][l], acc[idx(l, 0)]);
#pragma unroll
    for (int m = 1; m < NB; ++m) {
      legendre_row<NB>(m, G.z, one, r[(m - 1) & 1], r[m & 1]);
#pragma unroll
      for (int l = m; l < NB; ++l) {
        const float u = l == m ? g[l] : g[l] * r[m & 1][l];
        acc[idx(l, m)] = fmaf(u, C[m], acc[idx(l, m)]);
        acc[idx(l, -m)] = fmaf(u, Sn[m], acc[idx(l, -m)]);
      }
    }
  }
  // Coefficient i of the block is ((acc_0 + acc_1) + acc_2) + acc_3 over the
  // waves, in two exchanges of half the coefficients; each wave adds up every
  // fourth coefficient.
  constexpr int H = PairFwdHalf<NB>::H;
  const int w0 = __builtin_amdgcn_readfirstlane(wave);
  float* out = Fpart + (int64_t)by * N * P + p;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();  // the spheres (h = 0) or the previous half (h = 1) are no longer read
#pragma unroll
    for (int i = h * H; i < N && i < (h + 1) * H; ++i) X[wave][i - h * H][lane] = acc[i];
    __syncthreads();
    if (ok) {
#pragma unroll
      for (int b = h * H; b < N && b < (h + 1) * H; b += SHV_WAVES_PER_BLOCK) {
        const int i = b + w0;
        if (i < N && i < (h + 1) * H) {
          float v = X[0][i - h * H][lane];
#pragma unroll
          for (int w = 1; w < SHV_WAVES_PER_BLOCK; ++w) v += X[w][i - h * H][lane];
          out[(int64_t)i * P] = v;
        }
      }
    }
  }
  // Side job for the fused render path, spread over the first chunk's blocks:
  // the lit transfer matrix M(L), needed by the shading that follows in
  // stream order.
  if (M && by == 0) build_M_range<NB>(L, M, (int)(m_idx * SHV_BLOCK) + threadIdx.x, (int)(m_count * SHV_BLOCK));
}

template <int NB>
__global__ __launch_bounds__(SHV_BLOCK) void k_pair_fwd(const float* __restrict__ pts, int64_t P,
                                                        const float4* __restrict__ sph, int S, int chunk,
                                                        float* __restrict__ Fpart, const float* __restrict__ L,
                                                        float* __restrict__ M) {
  __shared__ PairFwdShared<NB> sh;
  pair_fwd_item<NB>(pts, P, sph, S, chunk, Fpart, L, M, blockIdx.x, blockIdx.y, blockIdx.x, gridDim.x, sh);
}

struct PairBwdShared {
  float4 sph[SHV_MAX_CHUNK];
  float4 red[SHV_MAX_CHUNK];
  float gpx_w[SHV_WAVES_PER_BLOCK - 1][3][64];
};

// v, computed here: a select between v and a constant does not become a branch
// around v's computation, which would split the loop body.
__device__ __forceinline__ float here(float v) {
  asm("" : "+v"(v));
  return v;
}

// Adjoint of one pair's term for the weights W_lm = dLoss/dF'_lm (and
// W0_l = ROW_0[l] W_l0, the weights of d p_l / dz in terms of rho_l^1): the
// cotangent of v = c - x (gvx, gvy, gvz) and of the radius (gr).
//
// With b_lm = W_lm C_m + W_l,-m S_m, the degrees' sums f_l = sum_m rho_l^m b_lm
// give dLoss/dt and h_l = sum_m (d rho_l^m / dz) b_lm the z derivative: one
// instruction each per term where separate sums over l for every order and
// both of cosine and sine took two, and no second set of weights.
//
// 1/t is wanted outside the sphere only.  A branch there is the faster form (64-scene
// batch: 262 us against 282 with selects at 4 bands, 517 against 522 at 6), but at 8 bands
// it splits the body, and the four waves per SIMD that 128 registers allow spill
// (762 us against 510).
template <int NB>
__device__ __forceinline__ void pair_adjoint(const PairGeom& G, float one, const float (&W)[NB * NB],
                                             const float (&W0)[NB], float& gvx, float& gvy, float& gvz, float& gr) {
  constexpr bool SELECT = NB == 8;
  float g[NB], C[NB], Sn[NB], r[2][NB], f[NB], h[NB];
  const float it = SELECT ? here(fast_rsqrt(G.t2)) : 0.0f;  // 1 / t
  const float t = !SELECT ? G.t : G.t2 > 0.0f ? G.t2 * it : 0.0f;
  cap_terms<NB>(t, G.u, G.s2, g);
  cs_powers<NB>(G.x, G.y, C, Sn);
  legendre_monic<NB>(G.z, r[0]);
  if constexpr (NB > 1) legendre_row<NB>(1, G.z, one, r[0], r[1]);
  f[0] = W[0];
#pragma unroll
  for (int l = 1; l < NB; ++l) {
    f[l] = W[idx(l, 0)] * r[0][l];
    h[l] = l == 1 ? W0[1] : W0[l] * r[1][l];
  }
  float Gx = 0.0f, Gy = 0.0f, Gz = 0.0f;
#pragma unroll
  for (int m = 1; m < NB; ++m) {
    const float(&rm)[NB] = r[m & 1];
    float(&rn)[NB] = r[(m + 1) & 1];
    legendre_row<NB>(m + 1, G.z, one, rm, rn);
    float Xc = 0.0f, Xs = 0.0f;
#pragma unroll
    for (int l = m; l < NB; ++l) {
      const float wc = W[idx(l, m)], ws = W[idx(l, -m)];
      const float b = fmaf(ws, Sn[m], wc * C[m]);
      f[l] = l == m ? f[l] + b : fmaf(rm[l], b, f[l]);
      if (l == m + 1) h[l] += b;
      else if (l > m) h[l] = fmaf((l - m) & 1 ? rn[l] : SHV_ROW_K[m] * rn[l], b, h[l]);
      const float v = l == m ? g[l] : g[l] * rm[l];
      Xc = fmaf(wc, v, Xc);
      Xs = fmaf(ws, v, Xs);
    }
    const float fm = (float)m;
    if (m == 1) {
      Gx = Xc;
      Gy = Xs;
    } else {
      const float mc = fm * C[m - 1], ms = fm * Sn[m - 1];
      Gx = fmaf(Xc, mc, fmaf(Xs, ms, Gx));
      Gy = fmaf(Xs, mc, fmaf(-Xc, ms, Gy));
    }
  }
  float p[NB];
  legendre_monic<NB>(t, p);
  float Gt = -f[0];  // d a_l / dt = -(l + 1) p_l
#pragma unroll
  for (int l = 1; l < NB; ++l) {
    Gz = fmaf(g[l], h[l], Gz);
    Gt = fmaf(-(float)(l + 1), p[l] * f[l], Gt);
  }
  // chain rule: s = v/|v| (tangential part / |v|), t(|v|, r)
  const float sd = fmaf(Gx, G.x, fmaf(Gy, G.y, Gz * G.z));
  gvx = (Gx - sd * G.x) * G.inv;
  gvy = (Gy - sd * G.y) * G.inv;
  gvz = (Gz - sd * G.z) * G.inv;
  // dLoss/dt * (-dt/dr); a receiver inside the sphere (t = 0) has none
  float k = 0.0f;
  if constexpr (SELECT) {
    const float ks = here((Gt * G.rs) * (it * G.inv));
    k = G.t2 > 0.0f ? ks : 0.0f;
  } else if (G.t > 0.0f) {
    k = (Gt * G.rs) * (fast_rcp(G.t) * G.inv);
  }
  const float kd = k * G.rs;  // dLoss/dt * dt/d|v|
  gvx = fmaf(kd, G.x, gvx);
  gvy = fmaf(kd, G.y, gvy);
  gvz = fmaf(kd, G.z, gvz);
  gr = -k;
}

template <int NB>
__device__ __forceinline__ void pair_bwd_item(const float* __restrict__ Wg, const float* __restrict__ pts, int64_t P,
                                              const float4* __restrict__ sph, int S, int chunk,
                                              float* __restrict__ gp_part, float4* __restrict__ gs_part, int64_t bx,
                                              int by, PairBwdShared& sh) {
  constexpr int N = NB * NB;
  auto& red = sh.red;
  auto& gpx_w = sh.gpx_w;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t p = bx * 64 + lane;
  const bool ok = p < P;
  const int s0 = by * chunk;
  const int s1 = min(S, s0 + chunk);
  const int64_t q = ok ? p : 0;  // valid receiver for the loads of tail lanes
  const float px = sel0(ok, pts[q]);
  const float py = sel0(ok, pts[P + q]);
  const float pz = sel0(ok, pts[2 * P + q]);

  // Zero on tail lanes, so they contribute nothing to the sphere sums.
  float W[N], W0[NB];
#pragma unroll
  for (int i = 0; i < N; ++i) W[i] = sel0(ok, Wg[(int64_t)i * P + q]);
#pragma unroll
  for (int l = 0; l < NB; ++l) W0[l] = W[idx(l, 0)] * SHV_ROW_0[l];

  float gpx = 0.0f, gpy = 0.0f, gpz = 0.0f;
  for (int j = threadIdx.x; j < s1 - s0; j += SHV_BLOCK) sh.sph[j] = sph[s0 + j];
  __syncthreads();
  const float one = vector_one();
  for (int s = s0 + wave; s < s1; s += SHV_WAVES_PER_BLOCK) {
    const PairGeom G = pair_geom(px, py, pz, sh.sph[s - s0]);
    float gvx, gvy, gvz, gr;
    pair_adjoint<NB>(G, one, W, W0, gvx, gvy, gvz, gr);
    gpx -= gvx;
    gpy -= gvy;
    gpz -= gvz;
    const float tot = wave_sum4(gvx, gvy, gvz, gr);  // total of (gvx, gvy, gvz, gr)[lane / 16]
    if ((lane & 15) == 15) reinterpret_cast<float*>(red)[(s - s0) * 4 + (lane >> 4)] = tot;  // one wave per sphere
  }
  if (wave > 0) {
    gpx_w[wave - 1][0][lane] = gpx;
    gpx_w[wave - 1][1][lane] = gpy;
    gpx_w[wave - 1][2][lane] = gpz;
  }
  __syncthreads();
  if (wave == 0 && ok) {
#pragma unroll
    for (int w = 0; w < SHV_WAVES_PER_BLOCK - 1; ++w) {
      gpx += gpx_w[w][0][lane];
      gpy += gpx_w[w][1][lane];
      gpz += gpx_w[w][2][lane];
    }
    float* out = gp_part + (int64_t)by * 3 * P + p;
    out[0] = gpx;
    out[P] = gpy;
    out[2 * P] = gpz;
  }
  for (int j = threadIdx.x; j < s1 - s0; j += SHV_BLOCK) gs_part[bx * S + s0 + j] = red[j];
}

template <int NB>
__global__ __launch_bounds__(SHV_BLOCK, NB == 8 ? 4 : 1) void k_pair_bwd(const float* __restrict__ Wg, const float* __restrict__ pts,
                                                        int64_t P, const float4* __restrict__ sph, int S, int chunk,
                                                        float* __restrict__ gp_part, float4* __restrict__ gs_part) {
  __shared__ PairBwdShared sh;
  pair_bwd_item<NB>(Wg, pts, P, sph, S, chunk, gp_part, gs_part, blockIdx.x, blockIdx.y, sh);
}

// ---------------------------------------------------------------------------
// Launchers for one band count (instantiated per band count in shv_nb.hip).

template <int NB>
hipError_t pair_fwd_nb(const float* pts, int64_t P, const float* sph, int S, Split sp, float* Fpart,
                       const float* light, float* M, hipStream_t st) {
  dim3 grid((unsigned)pair_blocks(P), (unsigned)sp.nchunks);
  k_pair_fwd<NB><<<grid, SHV_BLOCK, 0, st>>>(pts, P, (const float4*)sph, S, sp.chunk, Fpart, light, M);
  return hipGetLastError();
}

template <int NB>
hipError_t pair_bwd_nb(const float* W, const float* pts, int64_t P, const float* sph, int S, Split sp, float* gp_part,
                       float* gs_part, hipStream_t st) {
  dim3 grid((unsigned)pair_blocks(P), (unsigned)sp.nchunks);
  k_pair_bwd<NB><<<grid, SHV_BLOCK, 0, st>>>(W, pts, P, (const float4*)sph, S, sp.chunk, gp_part, (float4*)gs_part);
  return hipGetLastError();
}

// Batched pair phases over the scenes with NB bands, one block per item.
template <int NB>
__global__ __launch_bounds__(SHV_BLOCK) void k_batch_pair_fwd(const char* __restrict__ table) {
  __shared__ PairFwdShared<NB> sh;
  const BatchView v(table);
  const int64_t item = blockIdx.x;
  if (item >= v.h->total_pair_f[NB]) return;
  const BatchScene S = in_global(v.scene_of_pair_fwd(NB, item));
  const int64_t local = item - S.off_pair_f;
  const int64_t tile = local % S.range_tiles;
  const int by = (int)(local / S.range_tiles);
  pair_fwd_item<NB>(S.points, S.P, reinterpret_cast<const float4*>(S.spheres), (int)S.S, S.chunk_f, S.Fpart, S.light,
                    S.M, S.tile0 + tile, by, tile, S.range_tiles, sh);
}

template <int NB>
__global__ __launch_bounds__(SHV_BLOCK, NB == 8 ? 4 : 1) void k_batch_pair_bwd(const char* __restrict__ table) {
  __shared__ PairBwdShared sh;
  const BatchView v(table);
  const int64_t item = blockIdx.x;
  if (item >= v.h->total_pair_b[NB]) return;
  const BatchScene S = in_global(v.scene_of_pair_bwd(NB, item));
  if (!S.grad_radiance || (!S.grad_points && !S.grad_spheres)) return;  // uniform: nothing to do
  const int64_t local = item - S.off_pair_b;
  const int64_t bx = S.tile0 + local % S.range_tiles;
  const int by = (int)(local / S.range_tiles);
  pair_bwd_item<NB>(S.W, S.points, S.P, reinterpret_cast<const float4*>(S.spheres), (int)S.S, S.chunk_b, S.gp,
                    reinterpret_cast<float4*>(S.gs), bx, by, sh);
}

template <int NB>
hipError_t batch_pair_fwd_nb(const void* table, int64_t blocks, hipStream_t st) {
  k_batch_pair_fwd<NB><<<(unsigned)blocks, SHV_BLOCK, 0, st>>>((const char*)table);
  return hipGetLastError();
}

template <int NB>
hipError_t batch_pair_bwd_nb(const void* table, int64_t blocks, hipStream_t st) {
  k_batch_pair_bwd<NB><<<(unsigned)blocks, SHV_BLOCK, 0, st>>>((const char*)table);
  return hipGetLastError();
}

}  // namespace shv
