// Compressed passes that take and leave deferred weight updates (paper
// section 2: eq. (1) back-propagation and eq. (3) forward projection over one
// window of the random pixel order, eqs. (4)-(6) of the previous pass at the
// start): every compressed pass of an FP32 job with separable full-grid
// passes (N <= kDeferMaxSpots) or of a mixed job of one spot unit per wave.
//
// The arithmetic and the order of every sum are those of the per-pixel pass
// (k_pass_batch, k_pass_mx), so the results are its results bit for bit.
//
// Bound.  One hologram at 1152^2, N = 100, c = 1/16 (1296 tiles, five per
// compute unit): a chain of about 4 us (launch, the reads of state and totals,
// the update) in front of about 5 us of vector issue (38 cycles per 64 pairs
// back, 44 forward), and the additions at the end, which up to 64 spots bound
// the pass.  What this form takes off the per-pixel pass with deferred updates:
// the descriptor and job reads in front of everything else (arguments in
// registers), the totals' trips to memory (plain loads, shared in the L2), one
// of the tile's barriers with the normalisation of all four waves' pixels by
// one wave, half of the addition phase (one component per thread instead of
// two), 14 VGPRs (62 instead of 76: eight waves per SIMD instead of six), the
// ends of the blocks one after another (wave priorities that fall along the
// tile), and in large launches the starts of all but one tile in several and
// the idle lanes of the forward phase.  Hologram time, before and after: 1152^2,
// N = 100: 479 to 345 us (pass 14.2 to 10.1 us); 1920 x 1152 under the pupil, N =
// 52, c = 1/8: 442 to 251 us; N = 300, c = 1/16: 1249 to 870 us (no hand-off, no
// update in the tail); mixed, N = 100: 500 to 362 us; 32 holograms of 1152^2 per
// batch: 8.62 to 5.66 ms; 64 mixed ones 19.0 to 11.7 ms.  (The full-grid passes'
// own gains are in these.)
#include <math.h>

#include "device_common.hpp"
#include "device_math.hpp"
#include "kernels.hpp"
#include "pass_tail.hpp"
#include "pixel_pass.hpp"

namespace hg {

namespace {

// What the start of a pass reads, uniform across the block.
struct PassStart {
  const SpotRec* st;               // spot state before the previous pass's update
  const unsigned long long* tot;   // the previous pass's total set (null: no update)
  const int32_t* perm;
  int start, P, count, N, sub, W, H;
  uint32_t div_m;                  // row_divisor(W)
  int div_sh;
};

__device__ __forceinline__ int32_t window_pixel(const PassStart& h, int q) {
  uint32_t k = (uint32_t)h.start + (uint32_t)q;  // below 2 P <= 2^27
  if (k >= (uint32_t)h.P) k -= (uint32_t)h.P;
  return as_global(h.perm)[k];
}
__device__ __forceinline__ PixCoord coord_of(const PassStart& h, int32_t p) {
  return pixel_coord(p, h.W, h.H, h.div_m, h.div_sh);
}

// Phase 2 of 33 ... 256 spots by chains.  A unit of the per-pixel pass sums
// its slice's pixels in two chains, the even and the odd ones (its 64 lanes are
// 64 spots, so the last chunk of N spots leaves lanes idle: 28 of 128 at N =
// 100, a whole wave's work at N = 150).  Here the lanes of a wave are the 2^lgG
// chains of all slices times 64 >> lgG spots: the same chains of the same
// pixels in the same order, in ceil(N / (64 >> lgG)) <= 8 rounds, of which a wave
// takes one or two (two share the reads of the pixels).  For launches that
// fill the chip several times over, where the vector issue bounds the pass: 64
// mixed holograms of 8 to 200 spots 12.89 to 12.08 ms, 32 of 100 spots 5.75 to
// 5.65 ms.  One hologram's pass ends with its slowest wave, whose share of the
// pixels does not get smaller, and the form's 70 VGPRs hold seven blocks per
// compute unit instead of eight (1920 x 1152, N = 52: 265 to 279 us): there
// the units stay.
struct ChainMap {
  int lgL;     // lanes (spots) per chain 2^lgL = 8, 16 or 32: also its pixels
  int lgS;     // slices 2^lgS (two chains each)
  int rounds;  // ceil(N / 2^lgL)
  int stride;  // spots per chain in the table of sums
};
__device__ __forceinline__ ChainMap chain_map(int N) {
  ChainMap m;
  m.lgL = N <= 64 ? 3 : N <= 128 ? 4 : 5;
  m.lgS = 5 - m.lgL;
  m.rounds = (N + (1 << m.lgL) - 1) >> m.lgL;
  m.stride = 8 << m.lgL;
  return m;
}
template <int K>
__device__ __forceinline__ void chain_rounds(int N, const ChainMap& m, int round, int lane,
                                             const SpotRec* recs, const float4* px,
                                             const float* pui, float2* red) {
  const int L = 1 << m.lgL, c = lane >> m.lgL, g = lane & (L - 1);
  // chain c: pixels of slice c / 2 (2 L of them) of parity c % 2
  const int p0 = ((c >> 1) << (m.lgL + 1)) + (c & 1);
  float cx[K], cy[K], cz[K], vr[K], vi[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int n = ((round + k * kWaves) << m.lgL) + g;
    cx[k] = cy[k] = cz[k] = vr[k] = vi[k] = 0.f;
    if (n < N) {
      cx[k] = recs[n].cx;
      cy[k] = recs[n].cy;
      cz[k] = recs[n].cz;
    }
  }
  const float4* q = px + p0;
  const float* w = pui + p0;
  for (int i = 0; i < L; i += 2, q += 4, w += 4) {
    const float4 a0 = q[0], a1 = q[2];
    const float b0 = w[0], b1 = w[2];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      forward_term(cx[k], cy[k], cz[k], a0, b0, vr[k], vi[k]);
      forward_term(cx[k], cy[k], cz[k], a1, b1, vr[k], vi[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k)
    red[c * m.stride + ((round + k * kWaves) << m.lgL) + g] = make_float2(vr[k], vi[k]);
}
__device__ __forceinline__ void forward_chains(int N, const ChainMap& m, int role, int lane,
                                               const SpotRec* recs, const float4* px,
                                               const float* pui, float2* red) {
  static_assert(kWaves == 4, "at most two of eight rounds per wave");
  if (role + kWaves < m.rounds) chain_rounds<2>(N, m, role, lane, recs, px, pui, red);
  else chain_rounds<1>(N, m, role, lane, recs, px, pui, red);  // (five rounds at least)
}

// One pass of one job.  MAXU: spot units per wave (1: N <= 256, 2: N <= 512).
//
// A block takes its tiles of 64 pixels in turn.  Per 64 pixels:
//  phase 1  lane = pixel, wave w adds the spots [w N/4, (w+1) N/4); the four
//           shares meet in LDS (the one barrier of the tile's arithmetic);
//  u        every wave adds the shares of all 64 pixels in wave order,
//           normalises, and keeps u in its own LDS rows: no wave waits for
//           another's normalisation, which runs at the same time on the four
//           SIMDs;
//  phase 2  lanes = spots over the wave's pixels, as in the per-pixel pass.
// Then each component of the tile's sums is formed by one thread and added to
// the pass's total set, re and im in neighbouring lanes.
template <int MAXU, bool MX, bool CHAINS>
__device__ __forceinline__ void defer_tiles(const PassStart& h, const PassPlan& plan, int lb,
                                            int tot_row, unsigned long long* acc, float ill_a,
                                            const SpotRec* recs, PixCoord c) {
  __shared__ float2 sw[2][kWaves][kTile];
  __shared__ float4 px[kWaves][kTile];
  __shared__ float pui[kWaves][kTile];
  // sums of the units (64 lanes each), or of the chains (cl.stride spots each).
  // With two units per wave they take the wave's own pixel rows, which it has
  // read by then: 25.6 KB of LDS instead of 29.7, six blocks per compute unit
  // instead of five (1920 x 1152, N = 300: 903 to 874 us per hologram).
  __shared__ float2 red_own[MAXU > 1 ? 1 : kWaves * (CHAINS ? 2 : 1) * 64];
  float2* red = MAXU > 1 ? reinterpret_cast<float2*>(&px[0][0]) : red_own;
  static_assert(MAXU <= 2 && sizeof(px) == kWaves * 2 * 64 * sizeof(float2), "two units per row");
  auto unit_at = [](int u) { return MAXU > 1 ? 128 * (u & (kWaves - 1)) + 64 * (u / kWaves) : 64 * u; };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int N = h.N;
  const LaneMap lm = lane_map(N);
  const int Lg = 1 << lm.lgL, R = 64 >> lm.lgL, S = 1 << lm.lgS;
  const int g = lane & (Lg - 1), r = lane >> lm.lgL;
  auto unit_rec = [&](int u) {  // cx, cy, cz of this lane's spot in unit u
    const int n = ((u >> lm.lgS) << lm.lgL) + g;
    if (u >= lm.U || n >= N) return make_float3(0.f, 0.f, 0.f);
    return make_float3(recs[n].cx, recs[n].cy, recs[n].cz);
  };
  float3 rec[MAXU];
#pragma unroll
  for (int k = 0; k < MAXU; ++k)
    if (!CHAINS) rec[k] = unit_rec(wave + k * kWaves);
  const int n_lo = (int)((unsigned)(wave * N) / kWaves);
  const int n_hi = (int)((unsigned)((wave + 1) * N) / kWaves);
  const double scale = ldexp(1.0, plan.shift);
  // (parts of one tile add up between the chains: those stay with the units)
  const bool chains = CHAINS && N > 32 && plan.sub == 1;
  const ChainMap cl = chain_map(N);
  // The oldest wave of a SIMD issues first, so the blocks of a compute unit
  // finish one after another, and the last ones run alone, where a wave issues
  // at half the rate.  Priorities that fall along the tile keep the blocks
  // level instead: all of them up to 256 spots, the last four of a compute
  // unit in mixed precision, the last six (as many as fit at once) beyond 256
  // spots (N = 300: without 920, with four 880, with six 874 us per hologram).
  // 1152^2, N = 100: 365 to 346 us, mixed 371 to 362 us; N = 200, 2040 tiles 22.0 to
  // 21.2 us; N = 512 50.5 to 48.8 us.
  // In launches of several tiles per block the blocks' phases interleave the
  // better for it: 32 such holograms 5.94 to 5.71 ms, 64 mixed ones 12.2 to 11.8
  // ms.  Up to 64 spots the additions at the blocks' ends bound the pass, and
  // even ends crowd them (N = 52, 2040 tiles: 9.0 to 10.7 us; ten holograms, two
  // tiles per block, N = 16: 31.4 to 32.2 us a round): there only launches of many
  // tiles per block gain (eight, N = 52: 111 to 106 us; five, served: none).
  const bool paced = N > 64 || (CHAINS && plan.tiles >= 6 * plan.blocks);
  const bool late = paced && (CHAINS || (MAXU == 1 && !MX) || lb + (MAXU > 1 ? 6 : 4) * 256 >= plan.blocks);
  int turn = 0;  // which waves take the odd rounds: in turn over the block's tiles
  // this thread's components of the tiles' sums (x = threadIdx.x + i kBlock)
  constexpr int kSums = 2 * MAXU;  // 2 N <= kSums kBlock
  unsigned long long sums[kSums];
#pragma unroll
  for (int i = 0; i < kSums; ++i) sums[i] = 0ull;
  // the pixel index of the next 64 pixels is requested before the arithmetic
  // of the current ones
  int buf = 0;
  int32_t next = 0;
  for (int tile = lb; tile < plan.tiles; tile += plan.blocks) {
    float vr[MAXU], vi[MAXU];
#pragma unroll
    for (int k = 0; k < MAXU; ++k) vr[k] = vi[k] = 0.f;
    for (int st = 0; st < plan.sub; ++st) {
      if (paced) __builtin_amdgcn_s_setprio(2);
      const int32_t q = (tile * plan.sub + st) * kTile + lane;
      const bool valid = q < h.count;
      if (tile != lb || st != 0) c = coord_of(h, next);
      if (!valid) c = PixCoord{0.f, 0.f, 0.f, 0};
      const int32_t qn = (st + 1 < plan.sub ? q : ((tile + plan.blocks) * plan.sub - 1) * kTile + lane) + kTile;
      next = qn < h.count ? window_pixel(h, qn) : 0;
      sw[buf][wave][lane] =
          MX ? backprop_field_mx_lds(recs, n_lo, n_hi, c) : backprop_field_lds(recs, n_lo, n_hi, c);
      if (late) __builtin_amdgcn_s_setprio(1);
      __syncthreads();
      {
        float4 rec = make_float4(0.f, 0.f, 0.f, 0.f);
        float ui = 0.f;
        if (valid) {
          float2 S = sw[buf][0][lane];
#pragma unroll
          for (int w = 1; w < kWaves; ++w) {
            S.x += sw[buf][w][lane].x;
            S.y += sw[buf][w][lane].y;
          }
          float ur;
          unit_field(S, ur, ui);
          if (ill_a > 0.f) {
            const float wt = pupil_weight(c.Qi, c.Q, -1, ill_a);
            ur *= wt;
            ui *= wt;
          }
          rec = make_float4(c.Lx, c.Ly, c.Q, ur);
        }
        px[wave][lane] = rec;
        pui[wave][lane] = ui;
      }
      // (the wave's own rows: its LDS accesses complete in order)
      __builtin_amdgcn_wave_barrier();
      if (chains) {
        const int role = (wave + turn) & (kWaves - 1);
        forward_chains(h.N, cl, role, lane, recs, px[wave], pui[wave], red);
      } else {
#pragma unroll
        for (int k = 0; k < MAXU; ++k) {
          const int u = wave + k * kWaves;
          if (u >= lm.U) continue;
          const float3 q = CHAINS ? unit_rec(u) : rec[k];
          // (the order of the sums goes by the job's own unit count, also
          // where it shares the launch with jobs of more spots)
          if (MAXU == 1 || lm.U <= kWaves)
            forward_unit<true>(lm, u, r, q.x, q.y, q.z, px[wave], pui[wave], vr[k], vi[k]);
          else
            forward_unit<false>(lm, u, r, q.x, q.y, q.z, px[wave], pui[wave], vr[k], vi[k]);
        }
      }
      buf ^= 1;  // the next shares go to the other rows: one barrier is enough
    }
    if (!chains) {
      if (MAXU > 1) asm volatile("" ::: "memory");  // the rows are read before they are rewritten
#pragma unroll
      for (int k = 0; k < MAXU; ++k) {
        const int u = wave + k * kWaves;
        if (u < lm.U) red[unit_at(u) + lane] = make_float2(vr[k], vi[k]);
      }
    }
    if (paced) __builtin_amdgcn_s_setprio(0);
    turn += 1;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSums; ++i) {
      const int x = threadIdx.x + i * kBlock;
      if (x >= 2 * N) break;
      const int n = x >> 1, part = x & 1;
      const int ch = n >> lm.lgL, gg = n & (Lg - 1);
      const int u0 = ch << lm.lgS;
      const float* row = reinterpret_cast<const float*>(red + gg) + part;
      float s = 0.f;
      if (chains) {  // the two chains of a slice, then the slices
        const float* q = reinterpret_cast<const float*>(red) + x;
        for (int sl = 0; sl < (1 << cl.lgS); ++sl)
          s += q[2 * cl.stride * (2 * sl)] + q[2 * cl.stride * (2 * sl + 1)];
      } else if (R == 1) {
        for (int sl = 0; sl < S; ++sl) s += row[2 * unit_at(u0 + sl)];
      } else {
        for (int sl = 0; sl < S; ++sl)
          for (int rr = 0; rr < R; ++rr) s += row[2 * (unit_at(u0 + sl) + (rr << lm.lgL))];
      }
      sums[i] += (unsigned long long)llrint((double)s * scale);
    }
    if (tile + plan.blocks < plan.tiles) __syncthreads();  // red is rewritten
  }
  const int rows = MAXU == 1 ? kAccRows : acc_rows(N);
  unsigned long long* out = acc + (tot_row * rows + lb % rows) * acc_row_words(N);
#pragma unroll
  for (int i = 0; i < kSums; ++i) {
    const int x = threadIdx.x + i * kBlock;
    if (x < 2 * N) atomicAdd(out + x, sums[i]);
  }
}

// One round of deferring passes.  With one pass in the launch its start comes
// as kernel arguments, the first fourteen dwords of which are in registers
// when the wave begins: the reads of the state, the totals and the pixel
// order then start without waiting for the descriptor and, after it, the job
// record (two memory round trips), and `jobs` is that job.  nss: N, the shift
// of the row division from bit 16, parts per tile from bit 21; wh: W, H from
// bit 15, bit 31 set with several passes (then only descs and jobs count and
// `start` is the number of passes).
template <int MAXU, bool MX, bool CHAINS>
__global__ __launch_bounds__(kBlock, MAXU > 1 ? 4 : 6) void k_pass_defer(
    const SpotRec* st, const unsigned long long* tot, const int32_t* perm, int32_t start, int32_t P,
    int32_t count, uint32_t nss, uint32_t wh, uint32_t div_m, const PassDesc* __restrict__ descs,
    const JobDev* __restrict__ jobs) {
  // the start runs ahead of the arithmetic of the blocks that share the SIMD:
  // a block that is late with its update is late at the end
  __builtin_amdgcn_s_setprio(3);
  constexpr int kMaxN = MAXU > 1 ? kDeferMaxSpots : kBlock;
  __shared__ SpotRec recs[kMaxN];
  PassStart h{st, tot, perm, start, P, count, (int)(nss & 0xffffu), (int)(nss >> 21),
              (int)(wh & 0x7fffu), (int)(wh >> 15 & 0x7fffu), div_m, (int)(nss >> 16 & 31u)};
  const PassDesc* dp = descs;
  const JobDev* jp = jobs;
  int lb = blockIdx.x;
  if (wh >> 31) {  // several passes: `start` is their number
    dp += find_desc(descs, start, blockIdx.x);
    jp += dp->job;
    lb -= dp->block_begin;
    h = PassStart{dp->pending ? dp->st_in : jp->sp,
                  dp->pending ? jp->acc + dp->prev_row * acc_set_words(jp->N)
                              : nullptr,
                  dp->ps.perm, (int)dp->ps.start, dp->ps.M, dp->ps.count, jp->N, dp->plan.sub,
                  jp->W, jp->H, jp->row_div.m, jp->row_div.sh};
  }
  const PassDesc& d = *dp;
  const JobDev& jb = *jp;
  // the pixel of this lane in the block's first 64, requested with the state
  const int q0 = lb * h.sub * kTile + (int)(threadIdx.x & 63);
  const int32_t p0 = q0 < h.count ? window_pixel(h, q0) : 0;
  // The same waves update in every block (and take the odd unit in every
  // block): consecutive blocks of a compute unit start on another of its SIMDs,
  // so the longer shares spread by themselves.  Moved on by one wave per block
  // they meet on one SIMD again (1920 x 1152, N = 52: 255 to 266 us; N = 300,
  // the units moved too: 942 to 1048 us).
  PixCoord c;
  if (h.tot) {
    PendingState<kMaxN> ps;
    ps.load(h.st, h.tot, h.N);
    c = coord_of(h, p0);
    ps.apply(jb, d, h.N, lb == 0, recs, nullptr);
  } else {
    c = coord_of(h, p0);
    const HG_GLOBAL float* src = as_global(reinterpret_cast<const float*>(h.st));
    float* dst = reinterpret_cast<float*>(recs);
    for (int k = threadIdx.x; k < (int)(sizeof(SpotRec) / sizeof(float)) * h.N; k += kBlock)
      dst[k] = src[k];
    __syncthreads();
  }
  __builtin_amdgcn_s_setprio(0);
  defer_tiles<MAXU, MX, CHAINS>(h, d.plan, lb, d.tot_row, jb.acc, jb.ill_a, recs, c);
}

}  // namespace

void launch_pass_defer(const JobDev* jobs, const PassDesc* descs, int ndesc, int total_blocks,
                       bool wide, bool mixed, bool large, const PassHead& head,
                       hipStream_t s) {
  if (ndesc <= 0 || total_blocks <= 0) return;
  const dim3 grid(total_blocks), block(kBlock);
  const JobDev* j = ndesc == 1 ? jobs + head.job : jobs;
  const uint32_t nss = (uint32_t)head.N | ((uint32_t)head.row_div.sh << 16) | ((uint32_t)head.sub << 21);
  const uint32_t wh = (uint32_t)head.W | ((uint32_t)head.H << 15) | (ndesc > 1 ? 0x80000000u : 0u);
  const int32_t start = ndesc > 1 ? ndesc : head.start;
#define HG_LAUNCH(U, M, C)                                                                       \
  hipLaunchKernelGGL((k_pass_defer<U, M, C>), grid, block, 0, s, head.st, head.tot, head.perm,   \
                     start, head.P, head.count, nss, wh, head.row_div.m, descs, j)
  if (wide) HG_LAUNCH(2, false, false);
  else if (mixed && large) HG_LAUNCH(1, true, true);
  else if (mixed) HG_LAUNCH(1, true, false);
  else if (large) HG_LAUNCH(1, false, true);
  else HG_LAUNCH(1, false, false);
#undef HG_LAUNCH
}

}  // namespace hg
