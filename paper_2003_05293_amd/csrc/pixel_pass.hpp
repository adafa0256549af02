// Parts of the per-pixel passes shared by their kernels: pixel coordinates,
// the back-propagation sums of one pixel (eq. 1) with the spot records in
// LDS, the normalised field, and the forward terms and sums of a wave's
// spots (eq. 3).  Every kernel takes the arithmetic and the order of the
// sums from here, so a hologram gives the same bits in all of them.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "device_common.hpp"
#include "device_math.hpp"
#include "kernels.hpp"

namespace hg {
namespace {

// Doubled integer offsets of pixel p from the grid centre and Q = Lx^2+Ly^2
// (also as an integer, for the aperture test).
struct PixCoord {
  float Lx, Ly, Q;
  int32_t Qi;
};

__device__ __forceinline__ PixCoord pixel_coord_ij(int32_t i, int32_t j, int W, int H) {
  const int32_t lx = 2 * i - (W - 1);
  const int32_t ly = 2 * j - (H - 1);
  PixCoord c;
  c.Lx = (float)lx;
  c.Ly = (float)ly;
  c.Qi = lx * lx + ly * ly;
  c.Q = (float)c.Qi;
  return c;
}
__device__ __forceinline__ PixCoord pixel_coord(int32_t p, int W, int H) {
  const int32_t j = p / W;
  return pixel_coord_ij(p - j * W, j, W, H);
}
// The same with the row from a multiplication: j = ((2 p + 1) m) >> (32 + sh), m
// and sh from row_divisor(W), exact for p < 2^26 (W, H <= 8192).
__device__ __forceinline__ PixCoord pixel_coord(int32_t p, int W, int H, uint32_t m, int sh) {
  const int32_t j = (int32_t)(__umulhi(2u * (uint32_t)p + 1u, m) >> sh);
  return pixel_coord_ij(p - j * W, j, W, H);
}

// The same sum with the spot records in LDS (pending and chained
// passes, whose records change at their start): the four records of a group
// are read together (every lane the same address: broadcast reads).
__device__ __forceinline__ float2 backprop_field_lds(const SpotRec* recs, int n0, int n1,
                                                     const PixCoord& c) {
  float sr = 0.f, si = 0.f;
  int n = n0;
  for (; n + 3 < n1; n += 4) {
    float4 q[4];
    float sA[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      q[k] = *reinterpret_cast<const float4*>(&recs[n + k].cx);
      sA[k] = recs[n + k].A;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float t = fmaf(q[k].x, c.Lx, fmaf(q[k].y, c.Ly, fmaf(q[k].z, c.Q, q[k].w)));
      float sn, cs;
      sincos_turns(t, sn, cs);
      sr = fmaf(sA[k], cs, sr);
      si = fmaf(sA[k], sn, si);
    }
  }
  for (; n < n1; ++n) {
    const float t =
        fmaf(recs[n].cx, c.Lx, fmaf(recs[n].cy, c.Ly, fmaf(recs[n].cz, c.Q, recs[n].th)));
    float sn, cs;
    sincos_turns(t, sn, cs);
    sr = fmaf(recs[n].A, cs, sr);
    si = fmaf(recs[n].A, sn, si);
  }
  return make_float2(sr, si);
}

// Mixed-precision back-propagation (eq. 1): the phase of each spot in FP32
// turns with theta folded in, t_n = phi_n(p) / 2 pi + theta_n, its cosine
// and sine from v_sin/v_cos; the two spots of a pair have their cosines,
// their sines and their amplitudes A_n rounded to FP16 and packed, and one
// FP16 dot product accumulated in FP32 (v_dot2_f32_f16) adds each part of
// the pair's terms A_n e^{i 2 pi t_n}: re += (cos_1, cos_2).(A_1, A_2),
// im += (sin_1, sin_2).(A_1, A_2).  A spot left without a partner is paired
// with a zero amplitude.
__device__ __forceinline__ void mx_pair(float t1, float a1, float t2, float a2, float& sr,
                                        float& si) {
  float sn1, cs1, sn2, cs2;
  sincos_turns(t1, sn1, cs1);
  sincos_turns(t2, sn2, cs2);
  const h2v_t a = to_h2(a1, a2);
  sr = __builtin_amdgcn_fdot2(to_h2(cs1, cs2), a, sr, false);
  si = __builtin_amdgcn_fdot2(to_h2(sn1, sn2), a, si, false);
}
__device__ __forceinline__ float turns_of(float cx, float cy, float cz, float th,
                                          const PixCoord& c) {
  return fmaf(cx, c.Lx, fmaf(cy, c.Ly, fmaf(cz, c.Q, th)));
}
// Records from LDS (a pending pass's updated state).
__device__ __forceinline__ float2 backprop_field_mx_lds(const SpotRec* recs, int n0, int n1,
                                                        const PixCoord& c) {
  float sr = 0.f, si = 0.f;
  int n = n0;
  for (; n + 3 < n1; n += 4) {
    float t[4], A[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float4 q = *reinterpret_cast<const float4*>(&recs[n + k].cx);
      t[k] = turns_of(q.x, q.y, q.z, q.w, c);
      A[k] = recs[n + k].A;
    }
    mx_pair(t[0], A[0], t[1], A[1], sr, si);
    mx_pair(t[2], A[2], t[3], A[3], sr, si);
  }
  for (; n + 1 < n1; n += 2)
    mx_pair(turns_of(recs[n].cx, recs[n].cy, recs[n].cz, recs[n].th, c), recs[n].A,
            turns_of(recs[n + 1].cx, recs[n + 1].cy, recs[n + 1].cz, recs[n + 1].th, c),
            recs[n + 1].A, sr, si);
  if (n < n1)
    mx_pair(turns_of(recs[n].cx, recs[n].cy, recs[n].cz, recs[n].th, c), recs[n].A, 0.f, 0.f,
            sr, si);
  return make_float2(sr, si);
}

// u = S / |S| (1 where S = 0).  The square sum is written as the fused form,
// so that every kernel rounds it alike.
__device__ __forceinline__ void unit_field(const float2& S, float& ur, float& ui) {
  const float m2 = fmaf(S.x, S.x, S.y * S.y);
  ur = 1.f;
  ui = 0.f;
  if (m2 > 0.f) {
    const float inv = rsqrtf(m2);
    ur = S.x * inv;
    ui = S.y * inv;
  }
}

__device__ __forceinline__ void forward_term(float cx, float cy, float cz, const float4& a,
                                             float ui, float& vr, float& vi) {
  const float t = fmaf(cx, a.x, fmaf(cy, a.y, cz * a.z));
  float sn, cs;
  sincos_turns(t, sn, cs);
  // u * conj(e^{i 2 pi t})
  vr = fmaf(a.w, cs, fmaf(ui, sn, vr));
  vi = fmaf(ui, cs, fmaf(-a.w, sn, vi));
}

// Spot-lane layout of phase 2 for N spots.  Every size but the chunk count
// is a power of two, kept as its logarithm.
struct LaneMap {
  int lgL;  // lanes per spot group 2^lgL (8, 16, 32 or 64); replicas 64 >> lgL
  int nch;  // spot chunks = ceil(N / lanes)
  int lgS;  // pixel slices per chunk 2^lgS (1, 2 or 4)
  int U;    // units = chunks * slices
};

__host__ __device__ inline LaneMap lane_map(int N) {
  LaneMap m;
  m.lgL = N <= 8 ? 3 : N <= 16 ? 4 : N <= 32 ? 5 : 6;
  m.nch = (N + (1 << m.lgL) - 1) >> m.lgL;
  static_assert(kWaves == 4, "slices of four waves");
  m.lgS = m.nch == 1 ? 2 : m.nch == 2 ? 1 : 0;
  m.U = m.nch << m.lgS;
  return m;
}

// Forward sums of unit u (its spot chunk and pixel slice) over 64 pixels:
// px = (Lx, Ly, Q, Re u), pui = Im u.  PAIRS (passes of one unit per wave):
// four pixels per step, read from LDS together, into two sums; with more
// units per wave the registers go to the units' sums.
template <bool PAIRS>
__device__ __forceinline__ void forward_unit(const LaneMap& lm, int u, int r, float cx, float cy,
                                             float cz, const float4* px, const float* pui,
                                             float& vr, float& vi) {
  static_assert(kTile == 64, "slices of a 64-pixel tile");
  const int sl = u & ((1 << lm.lgS) - 1), R = 64 >> lm.lgL;
  const int j0 = (sl << (6 - lm.lgS)) + r, j1 = (sl + 1) << (6 - lm.lgS);
  float ar = vr, ai = vi, br = 0.f, bi = 0.f;
  int j = j0;
  if (PAIRS && R == 1) {
    // one replica (r = 0): the pixel loop is uniform across the
    // wave, so its counter and the LDS addresses stay scalar
    int ju = __builtin_amdgcn_readfirstlane(j0);
    const int ju1 = __builtin_amdgcn_readfirstlane(j1);
    for (; ju + 3 < ju1; ju += 4) {
      const float4 p0 = px[ju], p1 = px[ju + 1], p2 = px[ju + 2], p3 = px[ju + 3];
      const float u0 = pui[ju], u1 = pui[ju + 1], u2 = pui[ju + 2], u3 = pui[ju + 3];
      forward_term(cx, cy, cz, p0, u0, ar, ai);
      forward_term(cx, cy, cz, p1, u1, br, bi);
      forward_term(cx, cy, cz, p2, u2, ar, ai);
      forward_term(cx, cy, cz, p3, u3, br, bi);
    }
    j = ju;
  } else if (PAIRS) {
    for (; j + 3 * R < j1; j += 4 * R) {
      const float4 p0 = px[j], p1 = px[j + R], p2 = px[j + 2 * R], p3 = px[j + 3 * R];
      const float u0 = pui[j], u1 = pui[j + R], u2 = pui[j + 2 * R],
                  u3 = pui[j + 3 * R];
      forward_term(cx, cy, cz, p0, u0, ar, ai);
      forward_term(cx, cy, cz, p1, u1, br, bi);
      forward_term(cx, cy, cz, p2, u2, ar, ai);
      forward_term(cx, cy, cz, p3, u3, br, bi);
    }
  }
  for (; j < j1; j += R) forward_term(cx, cy, cz, px[j], pui[j], ar, ai);
  vr = ar + br;
  vi = ai + bi;
}

}  // namespace
}  // namespace hg
