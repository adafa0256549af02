// Full-grid FP32 passes as separable products on the gfx950 matrix cores.
//
// With doubled pixel offsets the phase of eq. (2) splits into a part in the
// column and a part in the row: e^{i phi_n(i,j)} = F_n(i) G_n(j).  The
// back-propagated field of eq. (1) over the whole grid is then the complex
// matrix product S = B F with B_n(j) = C_n G_n(j), C_n = A_n e^{i theta_n},
// and the forward sums of eq. (3) over all pixels are
//   V_n = (1/M) sum_j conj(G_n(j)) T[j][n],  T = U conj(F)^T,  U = e^{i Phi}.
// A complex product is a real one with K = 2 Np, the real and imaginary parts
// of each spot (or pixel column) interleaved along K.  The factor tables are
// evaluated once per hologram in FP64 (the spots do not move); C_n comes from
// the state, or from the previous pass's deferred update, which a pending
// pass (and the final hologram) applies at its start.
//
// The final hologram Phi = arg(B F) runs on v_mfma_f32_16x16x4_f32 (FP32
// operands and sums).  The iteration's pass, whose products end in the mean
// over all pixels, runs on v_mfma_f32_16x16x32_f16 with every operand scaled to
// at most 2048 and split into a whole number and the half of the remainder, x =
// hi + lo (F from its FP64 value), B with the half of what those two leave over
// on top: rest hi + lo lo + lo hi + hi lo + hi hi for S, the last four for T,
// accumulated in FP32.  These products cost 5/16 and 4/16 of the FP32 ones.
//
// Why whole numbers: the unit adds the eight products of a lane group aligned to
// the largest of them and drops what lies below 2^-23 of that, towards zero
// (then it adds the four groups, rounding each time).  With floating high parts a
// weak spot beside a strong one thus came out short by up to 2^-24 of the strong
// amplitude, at every pixel alike.  Products of whole numbers up to 2048 and sums
// of eight of them are exact; those of the low parts lose 2^-35 of full scale.
// What is left, relative to full scale (the largest |C_n|, or 1 for F and u): hi +
// lo is off by up to 2^-24 (a third of that rms; for an FP32 number between 1/2 and
// 1: 2^-25), B by 2^-36.  Fields of one pass against 64 bits, error of a spot
// relative to its own field, rms, for amplitudes spread over 0, 1, 2, 3 and 5 decades (640 x
// 480, N = 100, 24 draws): 2.9, 4.2, 12, 44 and 99 e-8; FP32 products 2.9, 4.7, 15,
// 55 and 110 e-8; halves of the floating form 2.9, 4.3, 19, 106 and 252 e-8.
#include <math.h>

#include "device_common.hpp"
#include "device_math.hpp"
#include "kernels.hpp"
#include "operand_layout.hpp"
#include "pass_tail.hpp"

namespace hg {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));

constexpr int kSepCB = kSepTileW / 16;  // 16-column blocks per tile

// What the start of a pass reads, uniform across the block: as kernel
// arguments where one job has the launch (see k_pass_defer), else from its
// descriptor and job record.
struct SepStart {
  const SpotRec* st;              // state before the previous pass's update
  const unsigned long long* tot;  // the previous pass's total set (null: no update)
  const float2* ga;               // G by row
  const void* f;                  // F operand of the back-propagation
  int N, S16, W, H;
  int tx, ty, lb;                 // this block's tile
};
// nst: N, S16 from bit 16; wh: W, H from bit 15, bit 31 set with several
// jobs, whose number is then nst.
template <bool FINAL>
__device__ __forceinline__ SepStart sep_start(const SpotRec* st, const unsigned long long* tot,
                                              const float2* ga, const void* f, uint32_t nst,
                                              uint32_t wh, const SepDesc*& dp, const JobDev*& jp) {
  SepStart h{st, tot, ga, f, (int)(nst & 0xffffu), (int)(nst >> 16), (int)(wh & 0x7fffu),
             (int)(wh >> 15 & 0x7fffu), (int)blockIdx.x, (int)blockIdx.y, 0};
  if (wh >> 31) {
    dp += find_desc(dp, (int)nst, blockIdx.x);
    jp += dp->job;
    h.lb = (int)blockIdx.x - dp->block_begin;
    h.ty = h.lb / dp->tiles_x;
    h.tx = h.lb - h.ty * dp->tiles_x;
    h.st = dp->st_in;
    h.tot = dp->pending
                ? jp->acc + dp->prev_row * acc_set_words(jp->N)
                : nullptr;
    h.ga = jp->sepGa;
    h.f = FINAL ? (const void*)jp->sepFc : (const void*)jp->sepFs;
    h.N = jp->N;
    h.S16 = jp->mx_steps;
    h.W = jp->W;
    h.H = jp->H;
  } else {
    h.lb = h.ty * (int)gridDim.x + h.tx;
  }
  return h;
}

// C_n of the pass into cs [16 S16] (zero beyond N): the deferred update of
// the previous pass, formed as its tail would, or the state's coefficients.
// Ends with a block barrier.
__device__ __forceinline__ void stage_coef(const SepStart& h, const SepDesc& d, const JobDev& jb,
                                           SpotRec* recs, float2* cs) {
  if (h.tot) {
    PendingState<kPendMaxSpots> ps;
    ps.load(h.st, h.tot, h.N);
    for (int n = h.N + threadIdx.x; n < 16 * h.S16; n += kBlock) cs[n] = make_float2(0.f, 0.f);
    ps.apply(jb, d, h.N, h.lb == 0, recs, cs);
  } else {
    for (int n = threadIdx.x; n < 16 * h.S16; n += kBlock) {
      float2 c = make_float2(0.f, 0.f);
      if (n < h.N) {
        const HG_GLOBAL float* f = as_global(reinterpret_cast<const float*>(jb.coef + n));
        c = make_float2(f[0], f[1]);
      }
      cs[n] = c;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------ final hologram ---

__device__ __forceinline__ f4_t mfma4(float a, float b, const f4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int kSepSteps = 8;  // K-steps per load group

// Operands of kSepSteps K-steps of S = B F for one wave: G_n(row) of its
// rows and the F operand of the tile's 16-column blocks.  Loads of the
// next group are issued before the products of the current one.
struct BpOps {
  float2 ga[kSepSteps];
  float fc[kSepSteps][kSepCB];
};
__device__ __forceinline__ void bp_load(BpOps& o, const float2* Ga, const float* Fc, int rb, int tx,
                                        int s0, int KS, int lane) {
  static_assert(kSepSteps % 4 == 0, "groups of whole step quads");
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int h = 0; h < kSepSteps; h += 4) {
    // four steps of G (float2 each) in two 16-byte loads, four of each F
    // operand in one
    const HG_GLOBAL f4_t* gp = as_global(reinterpret_cast<const f4_t*>(
        Ga + ga_index4(rb, s0 + h, KS, lr + 16 * (lg >> 1))));
    const f4_t g01 = gp[0], g23 = gp[1];
    o.ga[h] = make_float2(g01[0], g01[1]);
    o.ga[h + 1] = make_float2(g01[2], g01[3]);
    o.ga[h + 2] = make_float2(g23[0], g23[1]);
    o.ga[h + 3] = make_float2(g23[2], g23[3]);
#pragma unroll
    for (int t = 0; t < kSepCB; ++t) {
      const f4_t f = as_global(reinterpret_cast<const f4_t*>(
          Fc + op_index4(kSepCB * tx + t, s0 + h, KS, lane)))[0];
      o.fc[h][t] = f[0];
      o.fc[h + 1][t] = f[1];
      o.fc[h + 2][t] = f[2];
      o.fc[h + 3][t] = f[3];
    }
  }
}
// A operand: part of B (real output: (Br, -Bi)) or of i B (imaginary
// output: (Bi, Br)) with B_n(row) = C_n G_n(row) formed in FP32.
__device__ __forceinline__ void bp_mma(const BpOps& o, const float2* cs, int s0, int lg, int part,
                                       f4_t* sr, f4_t* si) {
#pragma unroll
  for (int q = 0; q < kSepSteps; ++q) {
    const float2 c = cs[2 * (s0 + q) + (lg >> 1)];
    const float br = c.x * o.ga[q].x - c.y * o.ga[q].y, bi = c.x * o.ga[q].y + c.y * o.ga[q].x;
    const float ar = part ? -bi : br, ai = part ? br : bi;
#pragma unroll
    for (int t = 0; t < kSepCB; ++t) {
      sr[t] = mfma4(ar, o.fc[q][t], sr[t]);
      si[t] = mfma4(ai, o.fc[q][t], si[t]);
    }
  }
}

__global__ __launch_bounds__(kBlock, 3) void k_sep_final(
    const SpotRec* st, const unsigned long long* tot, const float2* ga, const float* f,
    uint32_t nst, uint32_t wh, const SepDesc* __restrict__ descs, const JobDev* __restrict__ jobs) {
  extern __shared__ float2 cs[];           // [Np] C_n = A_n e^{i theta_n}
  __shared__ SpotRec recs[kPendMaxSpots];  // pending: the updated records
  const SepDesc* dp = descs;
  const JobDev* jp = jobs;
  const SepStart h = sep_start<true>(st, tot, ga, f, nst, wh, dp, jp);
  const SepDesc& d = *dp;
  const JobDev& jb = *jp;
  const float* Fc = static_cast<const float*>(h.f);
  const int KS = 8 * h.S16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4, part = lg & 1;
  const int rb = 4 * h.ty + wave;
  const int row0 = 16 * rb, col0 = kSepTileW * h.tx;

  // S = B F, K = 2 Np in groups of kSepSteps steps (KS = 8 S16 is a
  // multiple of kSepSteps), the next group's operands loaded ahead.
  f4_t sr[kSepCB], si[kSepCB];
#pragma unroll
  for (int t = 0; t < kSepCB; ++t) sr[t] = si[t] = f4_t{0.f, 0.f, 0.f, 0.f};
  static_assert(kSepSteps == 8, "K-step groups of 8: KS = 8 S16");
  const int G = KS / kSepSteps;
  // three operand buffers: the loads run two groups ahead of the products;
  // the first two are requested before C_n is staged, so that the two
  // reads overlap
  BpOps P, Q, R;
  bp_load(P, h.ga, Fc, rb, h.tx, 0, KS, lane);
  if (G > 1) bp_load(Q, h.ga, Fc, rb, h.tx, kSepSteps, KS, lane);
  stage_coef(h, d, jb, recs, cs);
  for (int gi = 0; gi < G; gi += 3) {
    if (gi + 2 < G) bp_load(R, h.ga, Fc, rb, h.tx, (gi + 2) * kSepSteps, KS, lane);
    bp_mma(P, cs, gi * kSepSteps, lg, part, sr, si);
    if (gi + 1 < G) {
      if (gi + 3 < G) bp_load(P, h.ga, Fc, rb, h.tx, (gi + 3) * kSepSteps, KS, lane);
      bp_mma(Q, cs, (gi + 1) * kSepSteps, lg, part, sr, si);
    }
    if (gi + 2 < G) {
      if (gi + 4 < G) bp_load(Q, h.ga, Fc, rb, h.tx, (gi + 4) * kSepSteps, KS, lane);
      bp_mma(R, cs, (gi + 2) * kSepSteps, lg, part, sr, si);
    }
  }

  HG_GLOBAL float* out = as_global_mut(d.out);
#pragma unroll
  for (int t = 0; t < kSepCB; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 4 * lg + r, col = col0 + 16 * t + lr;
      if (row < h.H && col < h.W) {
        const float phi = atan2f(si[t][r], sr[t][r]);
        const int64_t p = (int64_t)row * h.W + col;
        out[p] = phi;
        // the SLM's gray image of the final hologram
        if (jb.gray) store_gray(jb.gray, p, jb.gray_bits, gray_level(phi, jb.lut, jb.lut_levels));
      }
    }
}

// ------------------------------------------------------- iteration pass ---

__device__ __forceinline__ f4_t mfma16(const u4_t& a, const u4_t& b, const f4_t& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, a),
                                                __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
}
// (x, y), at most 2048 in magnitude, as halves of whole numbers, of the
// remainders, and of what those leave over.
struct Split {
  uint32_t hi, lo, rest;
};
__device__ __forceinline__ Split split_pair(float x, float y) {
  Split s;
  const float xw = rintf(x), yw = rintf(y);
  float l[2];
  s.hi = whole_halves(xw, yw);
  s.lo = pack_halves(x - xw, y - yw, l);
  s.rest = h2_bits(fmaf(l[0], -1.f, x - xw), fmaf(l[1], -1.f, y - yw));
  return s;
}
// For half pairs (re, im) of z: the pair of -i z, (im, -re).
__device__ __forceinline__ u4_t times_minus_i(const u4_t& v) {
  u4_t r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = __builtin_rotateleft32(v[k], 16) ^ 0x80000000u;
  return r;
}
// For half pairs (br, -bi): (bi, br).
__device__ __forceinline__ u4_t times_i_conj(const u4_t& v) {
  u4_t r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = __builtin_rotateleft32(v[k], 16) ^ 0x00008000u;
  return r;
}

// Power of two s with s max_n |C_n| <= 2048 (and at least 724): then the parts
// of s B stay within 2048, and u = S / |S| does not depend on s.  Every wave
// forms it from the staged coefficients.
__device__ __forceinline__ float coef_scale(const float2* cs, int N, int lane) {
  float m = 0.f;
  for (int n = lane; n < N; n += 64) m = fmaxf(m, fmaxf(fabsf(cs[n].x), fabsf(cs[n].y)));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  const uint32_t bits = __builtin_bit_cast(uint32_t, m);
  int e = (int)(bits >> 23);  // biased exponent of the largest part
  // zero, subnormal, infinite or NaN: as they are
  if (e == 0 || e == 255) return 1.f;
  if ((bits & 0x7fffffu) >= 0x3504f3u) ++e;  // |C| <= sqrt(2) m may reach the next power
  const int se = 127 + 10 - (e - 127);       // 2^(10 - (e - 127))
  return __builtin_bit_cast(float, (uint32_t)(se < 1 ? 1 : se > 254 ? 254 : se) << 23);
}

// One K-step (16 spots) of S = B F for one wave: G_n(row) of its four spots
// per lane and the split F operand of the tile's 16-column blocks.
struct ItOps {
  f4_t g02, g13;               // G of spots 4 g, 4 g + 2 and 4 g + 1, 4 g + 3
  u4_t f[kSepCB][2];           // hi, lo
};
__device__ __forceinline__ void it_load(ItOps& o, const float2* Ga, const u4_t* Fs, int rb, int tx,
                                        int s, int S16, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
  const float2* gp = Ga + ga_index4(rb, 8 * s + 2 * lg, 8 * S16, lr);
  o.g02 = as_global(reinterpret_cast<const f4_t*>(gp))[0];
  o.g13 = as_global(reinterpret_cast<const f4_t*>(gp + 16 * 4))[0];
#pragma unroll
  for (int t = 0; t < kSepCB; ++t) {
    const HG_GLOBAL u4_t* fp = as_global(Fs) + 2 * fc_index(kSepCB * tx + t, s, S16, lane);
    o.f[t][0] = fp[0];
    o.f[t][1] = fp[1];
  }
}
// A operands (br, -bi) (real part) and (bi, br) (imaginary part), B = C G.
__device__ __forceinline__ void it_mma(const ItOps& o, const float2* cs, float scale, int s, int lg,
                                       f4_t* sr, f4_t* si) {
  const int n0 = 16 * s + 4 * lg;
  const float gx[4] = {o.g02[0], o.g13[0], o.g02[2], o.g13[2]};
  const float gy[4] = {o.g02[1], o.g13[1], o.g02[3], o.g13[3]};
  u4_t rh, rl, rm;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float cx = cs[n0 + q].x * scale, cy = cs[n0 + q].y * scale;
    const float br = fmaf(cx, gx[q], -cy * gy[q]), bi = fmaf(cx, gy[q], cy * gx[q]);
    const Split b = split_pair(br, -bi);
    rh[q] = b.hi;
    rl[q] = b.lo;
    rm[q] = b.rest;
  }
  const u4_t re[3] = {rm, rl, rh};
  const u4_t im[3] = {times_i_conj(rm), times_i_conj(rl), times_i_conj(rh)};
#pragma unroll
  for (int p = 0; p < 5; ++p) {  // rest hi, lo lo, lo hi, hi lo, hi hi
    const int k = (p + 1) / 2, l = p & 1;
#pragma unroll
    for (int t = 0; t < kSepCB; ++t) {
      sr[t] = mfma16(re[k], o.f[t][l], sr[t]);
      si[t] = mfma16(im[k], o.f[t][l], si[t]);
    }
  }
}

// The F operand of the forward product, spot l % 16 and columns 4 (l / 16) + q of
// a 16-column block, from the table of the back-propagation (column l % 16,
// spots 4 (l / 16) + q), for jobs without one of its own: lane l reads the four
// spots 4 (l % 16 / 4) + q of column 4 (l / 16) + l % 4, and the four lanes of a
// quad exchange rows and columns.  Costs 0.8 us per pass at 1000 x 777, N = 52 (10.8
// to 11.6 us), nothing measurable where blocks fill the chip.
__device__ __forceinline__ int quad_source(int lane) {
  return 4 * (lane >> 4) + (lane & 3) + 16 * ((lane & 15) >> 2);
}
template <int CTRL>
__device__ __forceinline__ uint32_t quad_perm(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ u4_t quad_transpose(const u4_t& v, int lane) {
  constexpr int kXor1 = 0xb1, kXor2 = 0x4e;  // lanes (1, 0, 3, 2) and (2, 3, 0, 1)
  const bool b0 = lane & 1, b1 = lane & 2;
  // (every lane takes part in an exchange: they stand outside the selections)
  const u4_t x = {quad_perm<kXor1>(v[1]), quad_perm<kXor1>(v[0]), quad_perm<kXor1>(v[3]),
                  quad_perm<kXor1>(v[2])};
  const u4_t a = {b0 ? x[0] : v[0], b0 ? v[1] : x[1], b0 ? x[2] : v[2], b0 ? v[3] : x[3]};
  const u4_t y = {quad_perm<kXor2>(a[2]), quad_perm<kXor2>(a[3]), quad_perm<kXor2>(a[0]),
                  quad_perm<kXor2>(a[1])};
  return u4_t{b1 ? y[0] : a[0], b1 ? y[1] : a[1], b1 ? a[2] : y[2], b1 ? a[3] : y[3]};
}

// T = U conj(F)^T for R 16-spot blocks starting at sb0 and the wave's 16
// rows, then the wave's partial V_n = sum_j conj(G_n(j)) T[j][n] of those
// spots into red (LDS).
template <int R, bool OWN_FN>
__device__ __forceinline__ void it_forward(const JobDev& jb, const u4_t* Fs, const u4_t (*ua)[2],
                                           const u4_t (*ub)[2], float2* red, int sb0, int rb,
                                           int tx, int S16, int CB, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
  const u4_t* Fn = reinterpret_cast<const u4_t*>(jb.sepFn);
  u4_t f[kSepCB][R][2];
#pragma unroll
  for (int t = 0; t < kSepCB; ++t)
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int cb = kSepCB * tx + t;
      const HG_GLOBAL u4_t* fp =
          OWN_FN ? as_global(Fn) + 2 * fn_index(sb0 + k, cb, CB, lane)
                 : as_global(Fs) + 2 * fc_index(cb, sb0 + k, S16, quad_source(lane));
      f[t][k][0] = fp[0];
      f[t][k][1] = fp[1];
    }
  // G of the V sums, requested with F (it does not depend on the products)
  f4_t gva[R], gvb[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int64_t gv = op_index(rb, sb0 + k, S16, lane) * 2;
    gva[k] = as_global(reinterpret_cast<const f4_t*>(jb.sepGv))[gv];
    gvb[k] = as_global(reinterpret_cast<const f4_t*>(jb.sepGv))[gv + 1];
  }
  f4_t tr[R], ti[R];
#pragma unroll
  for (int k = 0; k < R; ++k) tr[k] = ti[k] = f4_t{0.f, 0.f, 0.f, 0.f};
  if (!OWN_FN) {
#pragma unroll
    for (int t = 0; t < kSepCB; ++t)
#pragma unroll
      for (int k = 0; k < R; ++k) {
        f[t][k][0] = quad_transpose(f[t][k][0], lane);
        f[t][k][1] = quad_transpose(f[t][k][1], lane);
      }
  }
#pragma unroll
  for (int t = 0; t < kSepCB; ++t)
#pragma unroll
    for (int p = 0; p < 4; ++p)  // lo lo, lo hi, hi lo, hi hi
#pragma unroll
      for (int k = 0; k < R; ++k) {
        tr[k] = mfma16(ua[t][p < 2], f[t][k][(p & 1) == 0], tr[k]);
        ti[k] = mfma16(ub[t][p < 2], f[t][k][(p & 1) == 0], ti[k]);
      }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const f4_t g01 = gva[k], g23 = gvb[k];
    const float gr[4] = {g01[0], g01[2], g23[0], g23[2]};
    const float gi[4] = {g01[1], g01[3], g23[1], g23[3]};
    float vr = 0.f, vi = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      vr = fmaf(gr[r], tr[k][r], fmaf(gi[r], ti[k][r], vr));
      vi = fmaf(gr[r], ti[k][r], fmaf(-gi[r], tr[k][r], vi));
    }
    // the four row groups: rows of 16 lanes exchanged and added, re in the
    // first row, im in the second
    const float v = row_pair_sum(vr, vi);
    if (lg < 2) reinterpret_cast<float*>(red + 16 * (sb0 + k) % kSepRed + lr)[lg] = v;
  }
}

// Per 64 x 32 output tile, wave w owns 16 rows; nothing is shared between the
// waves but C_n until the tile's partial sums meet.
//
// Bound: at 1152^2, N = 100 (648 tiles, 2.5 per compute unit) the matrix cores
// need about 6 us (FP32 products: 18 us on the busiest SIMD), forming and
// splitting B about 3 us; the rest is the chain of launch, the pending update
// and the operand loads in front of them.  FP32 products with the descriptor
// read in front of the loads, and these split products with their start as
// arguments: 1152^2, N = 100: 33.4 and 18.5 us; 1000 x 777, N = 52: 15.6 and
// 10.8 us; 1920 x 1152, N = 300: 133 and 67 us; 32 holograms of 1152^2 in one
// launch: 717 and 460 us.  (Halves of the floating form without the products rest hi
// and lo lo: 16.0, 9.7, 59 and 416 us, less precise beside strong spots.)
// OWN_FN: the forward product has a table of its own.
template <bool OWN_FN>
__global__ __launch_bounds__(kBlock, 3) void k_sep_iter(
    const SpotRec* st, const unsigned long long* tot, const float2* ga, const void* f, uint32_t nst,
    uint32_t wh, const SepDesc* __restrict__ descs, const JobDev* __restrict__ jobs) {
  extern __shared__ float2 cs[];                         // [Np] C_n = A_n e^{i theta_n}
  __shared__ SpotRec recs[kPendMaxSpots];                // pending: the updated records
  // u of each wave's rows, split (hi and lo half pairs); rows of 36 words:
  // 16-byte reads of four columns at a time
  __shared__ uint32_t us[kWaves][2][16][kSepTileW + 4];
  __shared__ float2 red[kWaves][kSepRed];
  __shared__ int flag;
  const SepDesc* dp = descs;
  const JobDev* jp = jobs;
  const SepStart h = sep_start<false>(st, tot, ga, f, nst, wh, dp, jp);
  const SepDesc& d = *dp;
  const JobDev& jb = *jp;
  const u4_t* Fs = static_cast<const u4_t*>(h.f);
  const int W = h.W, H = h.H, N = h.N, S16 = h.S16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int rb = 4 * h.ty + wave;
  const int row0 = 16 * rb, col0 = kSepTileW * h.tx;

  // S = B F: the operands of the next two K-steps are on their way during a
  // step's products, the first two also while C_n is staged
  f4_t sr[kSepCB], si[kSepCB];
#pragma unroll
  for (int t = 0; t < kSepCB; ++t) sr[t] = si[t] = f4_t{0.f, 0.f, 0.f, 0.f};
  {
    ItOps P, Q, R;
    it_load(P, h.ga, Fs, rb, h.tx, 0, S16, lane);
    if (S16 > 1) it_load(Q, h.ga, Fs, rb, h.tx, 1, S16, lane);
    stage_coef(h, d, jb, recs, cs);
    const float scale = coef_scale(cs, N, lane);
    for (int s = 0; s < S16; s += 3) {
      if (s + 2 < S16) it_load(R, h.ga, Fs, rb, h.tx, s + 2, S16, lane);
      it_mma(P, cs, scale, s, lg, sr, si);
      if (s + 1 < S16) {
        if (s + 3 < S16) it_load(P, h.ga, Fs, rb, h.tx, s + 3, S16, lane);
        it_mma(Q, cs, scale, s + 1, lg, sr, si);
      }
      if (s + 2 < S16) {
        if (s + 4 < S16) it_load(Q, h.ga, Fs, rb, h.tx, s + 4, S16, lane);
        it_mma(R, cs, scale, s + 2, lg, sr, si);
      }
    }
  }

  // u = e^{i Phi} over the pupil (0 outside it and outside the grid),
  // weighted by the illumination, times kSplitScale and split, in the wave's
  // own LDS rows.
  const bool pupil = jb.ap_q >= 0 || jb.ill_a > 0.f;
#pragma unroll
  for (int t = 0; t < kSepCB; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = row0 + 4 * lg + r, col = col0 + 16 * t + lr;
      float ux = 0.f, uy = 0.f;
      if (row < H && col < W) {
        const float m2 = fmaf(sr[t][r], sr[t][r], si[t][r] * si[t][r]);
        ux = kSplitScale;
        if (m2 > 0.f) {
          const float inv = rsqrtf(m2) * kSplitScale;
          ux = sr[t][r] * inv;
          uy = si[t][r] * inv;
        }
        if (pupil) {
          const int32_t lx = 2 * col - (W - 1), ly = 2 * row - (H - 1);
          const int32_t Qi = lx * lx + ly * ly;
          const float wt = pupil_weight(Qi, (float)Qi, jb.ap_q, jb.ill_a);
          ux *= wt;
          uy *= wt;
        }
      }
      const Split u = split_pair(ux, uy);
      us[wave][0][4 * lg + r][16 * t + lr] = u.hi;
      us[wave][1][4 * lg + r][16 * t + lr] = u.lo;
    }
  // (the wave's own rows: its LDS accesses complete in order)
  __builtin_amdgcn_wave_barrier();
  u4_t ua[kSepCB][2], ub[kSepCB][2];  // u and -i u; hi, lo
#pragma unroll
  for (int t = 0; t < kSepCB; ++t)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      ua[t][p] = *reinterpret_cast<const u4_t*>(&us[wave][p][lr][16 * t + 4 * lg]);
      ub[t][p] = times_minus_i(ua[t][p]);
    }

  // T and the partial V in groups of four 16-spot blocks, then the rest; the
  // sums of up to kSepRed spots meet at a time, into the tile's group row, or,
  // when the pass defers its update, into a row of its total set (no counting:
  // the next launch reads the set)
  const int CB = jb.mx_cblocks;
  const int grp = h.lb / d.plan.group_size;
  unsigned long long* out =
      jb.acc + (d.defer ? (d.tot_row * acc_rows(N) + h.lb % acc_rows(N)) * acc_row_words(N)
                        : acc_group_at(N, grp));
  // T carries kSplitScale twice (exact powers of two)
  const double unit = ldexp(1.0, d.plan.shift - 2 * kSplitBits);
  for (int b0 = 0; b0 < S16; b0 += kSepRed / 16) {
    const int b1 = min(S16, b0 + kSepRed / 16);
    int sb = b0;
    for (; sb + 4 <= b1; sb += 4) it_forward<4, OWN_FN>(jb, Fs, ua, ub, red[wave], sb, rb, h.tx, S16, CB, lane);
    switch (b1 - sb) {
      case 3: it_forward<3, OWN_FN>(jb, Fs, ua, ub, red[wave], sb, rb, h.tx, S16, CB, lane); break;
      case 2: it_forward<2, OWN_FN>(jb, Fs, ua, ub, red[wave], sb, rb, h.tx, S16, CB, lane); break;
      case 1: it_forward<1, OWN_FN>(jb, Fs, ua, ub, red[wave], sb, rb, h.tx, S16, CB, lane); break;
      default: break;
    }
    __syncthreads();
    static_assert(2 * kSepRed <= kBlock, "one component per thread");
    const int x = 32 * b0 + (int)threadIdx.x;  // component of the sums
    if ((int)threadIdx.x < 2 * kSepRed && x < 2 * N) {
      const float* q = reinterpret_cast<const float*>(red[0]) + threadIdx.x;
      float v = q[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += q[2 * kSepRed * w];
      atomicAdd(out + x, (unsigned long long)llrint((double)v * unit));
    }
    if (b1 < S16) __syncthreads();  // red is rewritten
  }
  if (d.defer) return;

  __syncthreads();  // (every wave is past its use of cs)
  PassCtx a;
  a.sp = jb.sp;
  a.coef = jb.coef;
  a.N = N;
  a.W = W;
  a.H = H;
  a.ps = PixelSet{nullptr, nullptr, 0, W * H, W * H};
  a.phi = nullptr;
  a.plan = d.plan;
  a.lb = h.lb;
  a.partial = jb.partial;
  a.gpart = jb.gpart;
  a.acc = jb.acc;
  a.counters = jb.counters;
  a.inv_count = d.inv_count;
  a.V = d.V;
  a.status = jb.status;
  a.update = d.update;
  a.from_phi = 0;
  a.tot_row = d.tot_row;
  if (d.pending) {  // the update starts from the records in LDS
    a.recs = recs;
    a.pend_row = d.prev_row;
  }
  const int size = min(d.plan.group_size, d.plan.tiles - grp * d.plan.group_size);
  if (arrive_last(&jb.counters[grp * kCounterStride], (unsigned)size, &flag) &&
      tail_group(a, grp, &flag))
    tail_final(a, cs);  // the C_n table (Np >= N float2) is no longer read
}

}  // namespace

PassPlan plan_sep(int W, int H) {
  PassPlan p;
  p.tiles = ceil_div(W, kSepTileW) * ceil_div(H, kSepTileH);
  p.sub = 1;
  p.blocks = p.tiles;
  int gs = 1;
  while (gs * gs < p.blocks) ++gs;
  p.group_size = gs;
  p.ngroups = ceil_div(p.blocks, gs);
  p.shift = sum_shift((int64_t)W * H);
  return p;
}

void launch_sep_pass(const JobDev* jobs, const SepDesc* descs, int ndesc, int total_blocks,
                     bool final, int max_steps, const SepHead& head, hipStream_t s) {
  if (ndesc <= 0 || total_blocks <= 0) return;
  const size_t shmem = sizeof(float2) * 16 * (size_t)(max_steps > 0 ? max_steps : 1);
  const bool one = ndesc == 1;
  const dim3 grid = one ? dim3(head.tiles_x, head.tiles_y) : dim3(total_blocks);
  const JobDev* j = one ? jobs + head.job : jobs;
  const uint32_t nst = one ? (uint32_t)head.N | ((uint32_t)head.S16 << 16) : (uint32_t)ndesc;
  const uint32_t wh = (uint32_t)head.W | ((uint32_t)head.H << 15) | (one ? 0u : 0x80000000u);
  if (final)
    hipLaunchKernelGGL(k_sep_final, grid, dim3(kBlock), shmem, s, head.st, head.tot, head.ga,
                       head.fc, nst, wh, descs, j);
  else if (head.own_fn)
    hipLaunchKernelGGL(k_sep_iter<true>, grid, dim3(kBlock), shmem, s, head.st, head.tot, head.ga,
                       (const void*)head.fs, nst, wh, descs, j);
  else
    hipLaunchKernelGGL(k_sep_iter<false>, grid, dim3(kBlock), shmem, s, head.st, head.tot, head.ga,
                       (const void*)head.fs, nst, wh, descs, j);
}

}  // namespace hg
