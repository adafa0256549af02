// Hand-off of the FP32 passes: the per-block context, the exact fixed-point
// sums of the forward projection (eq. 3) and the weight update of eqs.
// (4)-(6), shared by the per-pixel and the separable kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "device_common.hpp"
#include "device_math.hpp"
#include "kernels.hpp"

namespace hg {
namespace {

// Everything one (virtual) block of a pass needs, uniform across the block.
struct PassCtx {
  SpotRec* sp;
  float2* coef;
  int N, W, H;
  PixelSet ps;
  const float* phi;
  PassPlan plan;
  int lb;  // this block within the pass
  float2* partial;
  double2* gpart;
  unsigned long long* acc;
  unsigned* counters;
  double inv_count;
  double2* V;
  int32_t* status;
  int update, from_phi;
  // pupil: forward terms weighted by the illumination (ill_a > 0), and
  // pixels outside the aperture dropped (ap_q >= 0: the whole-grid set)
  int32_t ap_q = -1;
  float ill_a = 0.f;
  // deferred updates (PassDesc): the total row of this pass's sums, whether
  // the pass stops after the group sums, and the previous pass's total row,
  // which the update clears (-1: none)
  int tot_row = 0;
  int defer = 0;
  int pend_row = -1;
  // chained launches and pending passes: the pass's spot state in LDS;
  // chained launches: the generation word to publish after the update
  int chain = 0;
  const SpotRec* recs = nullptr;
  unsigned* gen = nullptr;
  unsigned gen_next = 0;
};

// Device-scope copies of a spot record (read by the other blocks of a
// chained launch after the generation word says it is complete).
__device__ __forceinline__ void store_rec_dev(SpotRec* p, const SpotRec& r) {
  uint64_t w[4];
  __builtin_memcpy(w, &r, sizeof(w));
  HG_GLOBAL uint64_t* q = as_global_mut(reinterpret_cast<uint64_t*>(p));
#pragma unroll
  for (int i = 0; i < 4; ++i) __hip_atomic_store(q + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void load_recs_dev(const SpotRec* sp, int N, SpotRec* recs_lds) {
  const HG_GLOBAL uint64_t* q = as_global(reinterpret_cast<const uint64_t*>(sp));
  uint64_t* d = reinterpret_cast<uint64_t*>(recs_lds);
  for (int k = threadIdx.x; k < 4 * N; k += kBlock)
    d[k] = __hip_atomic_load(q + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exact sums.  Each tile's per-spot partial is rounded once to a 64-bit
// fixed-point integer (scale 2^shift, |sum over the pass| <= pixels, so no
// sum overflows) and added with device-scope integer atomics: integer
// addition is associative, so the sums do not depend on the order in which
// tiles, groups or blocks arrive.  Rows: the sets of pass totals (acc_rows(N)
// each), then the groups'.
__device__ __forceinline__ void acc_add(unsigned long long* row, int shift, int n, float2 v) {
  const double scale = ldexp(1.0, shift);
  unsigned long long* p = row + n * kAccSpotWords;
  atomicAdd(p, (unsigned long long)llrint((double)v.x * scale));
  atomicAdd(p + 1, (unsigned long long)llrint((double)v.y * scale));
}
__device__ __forceinline__ unsigned long long take_dev(unsigned long long* p) {
  HG_GLOBAL unsigned long long* q = as_global_mut(p);
  const unsigned long long v = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return v;
}

// Group g of tiles is complete: move its sums into the pass total (and clear
// them for the next pass), then count the group.  Returns true in the block
// that completes the last group.
__device__ bool tail_group(const PassCtx& a, int g, int* flag) {
  for (int k = threadIdx.x; k < 2 * a.N; k += kBlock) {
    const int64_t e = (int64_t)(k >> 1) * kAccSpotWords + (k & 1);  // spot k / 2, part k % 2
    const unsigned long long v = take_dev(a.acc + acc_group_at(a.N, g) + e);
    atomicAdd(a.acc + a.tot_row * acc_set_words(a.N) + e, v);
  }
  return arrive_last(&a.counters[a.plan.ngroups * kCounterStride], (unsigned)a.plan.ngroups, flag);
}

// The weight update of eqs. (4)-(6) in FP32: the one place that does this
// arithmetic, so that a deferred update gives the bits of an immediate one.
// A spot field enters as the FP64 mean of the exact sums rounded to FP32.
__device__ __forceinline__ float2 field32(double2 t) { return make_float2((float)t.x, (float)t.y); }
__device__ __forceinline__ float mag32(float2 v) { return sqrtf(fmaf(v.x, v.x, v.y * v.y)); }
// Sum over a wave, valid in lane 0, as the tree over lanes 32, 16, 8, 4, 2
// and 1 apart.  Halves and rows are exchanged by lane swaps, the lanes of a
// row by rotations: in every step the lane that is read holds the same bits
// as the one that many lanes above (the sums are symmetric), and no step
// goes through LDS.
__device__ __forceinline__ float swap_add(float x, bool rows) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = rows ? __builtin_amdgcn_permlane16_swap(u, u, false, false)
                      : __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// Sums of a and of b over the four rows of 16 lanes: a's in the first row,
// b's in the second.
__device__ __forceinline__ float row_pair_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                  __builtin_bit_cast(unsigned, b), false, false);
  // rows (a0 + a1, b0 + b1, a2 + a3, b2 + b3), then the halves
  return swap_add(__builtin_bit_cast(float, (unsigned)r[0]) +
                      __builtin_bit_cast(float, (unsigned)r[1]),
                  false);
}
template <int N>
__device__ __forceinline__ float ror_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                           0, __builtin_bit_cast(int, x), 0x120 + N, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_tree_sum(float x) {
  x = swap_add(x, false);
  x = swap_add(x, true);
  x = ror_add<8>(x);
  x = ror_add<4>(x);
  x = ror_add<2>(x);
  return ror_add<1>(x);
}
// mean_n |V_n| (eq. 4), the same in every thread of the block: thread t
// adds |V_n| for n = t, t + kBlock, ... in that order, starting from 0 (s
// is that thread sum); the thread sums are added in a fixed tree within
// each wave, then the wave sums in wave order.  Every thread must call it
// (it holds a block barrier).
__device__ __forceinline__ float block_mean_of(float s, int N) {
  const int t = threadIdx.x;
  __shared__ float wsum[kWaves];
  s = wave_tree_sum(s);
  if ((t & 63) == 0) wsum[t >> 6] = s;
  __syncthreads();
  float total = wsum[0];
  for (int w = 1; w < kWaves; ++w) total += wsum[w];
  return total / (float)N;
}
// The angle of v in turns.  A function of its own, never inlined: the
// library's atan2f carries a division of relaxed accuracy whose form depends
// on what the compiler merges it with, and the immediate and the deferred
// update, in whichever kernel, have to give the same bits.
__device__ __attribute__((noinline)) float arg_turns(float2 v) {
  return atan2f(v.y, v.x) * 0.15915494309189535f;
}
// false (record unchanged) where the weight would come out zero or not finite
__device__ __forceinline__ bool update_rec(SpotRec& r, float2 v, float mag, float mean) {
  const float w = r.w * (mean / mag);
  if (!(mag > 0.f) || !isfinite(w)) return false;
  r.w = w;
  r.A = w * r.a0;
  r.th = arg_turns(v);
  return true;
}

// Every group is complete: V_n = total / 2^shift / |Omega| (the total row is
// cleared for the next pass, and so are the counters); with a.update,
// eqs. (4)-(6): w_n <- w_n mean/|V_n|, theta_n <- arg V_n, A_n = a_n^0 w_n.
// vs: LDS room for N float2 (the spot fields in FP32, kept for the update:
// values other threads stored to memory are not read back, since a block
// of a chained launch may hold stale copies of them in its L1 cache).
// In a chained launch the passes' updates run in blocks on any XCD, and the
// XCDs' L2 caches write back independently: a plain store of C_n or V_n
// could leave an older pass's value dirty in one L2 and written back after
// the newer one, so there every state word goes out with device-scope
// stores (not left dirty in any L2).
__device__ void tail_final(const PassCtx& a, float2* vs) {
  const int N = a.N;
  const double inv = ldexp(1.0, -a.plan.shift) * a.inv_count;
  unsigned long long* tot = a.acc + a.tot_row * acc_set_words(N);
  float msum = 0.f;
  for (int n = threadIdx.x; n < N; n += kBlock) {
    const long long re = (long long)take_dev(tot + (int64_t)n * kAccSpotWords);
    const long long im = (long long)take_dev(tot + (int64_t)n * kAccSpotWords + 1);
    const double2 t = make_double2((double)re * inv, (double)im * inv);
    if (a.chain) store_dev(a.V + n, t);
    else a.V[n] = t;
    const float2 v = field32(t);
    vs[n] = v;
    msum += mag32(v);
  }
  // the previous pass's total set, which every block of this pass has read
  // before counting its tiles, is cleared
  if (a.pend_row >= 0) {
    HG_GLOBAL unsigned long long* q =
        as_global_mut(a.acc + a.pend_row * acc_set_words(N));
    for (int k = threadIdx.x; k < acc_set_words(N); k += kBlock)
      __hip_atomic_store(q + k, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // the counters are ready for the next pass (kernel end orders these
  // writes; in a chained launch, the generation word)
  for (int k = threadIdx.x; k <= a.plan.ngroups; k += kBlock) {
    if (a.chain)
      __hip_atomic_store(a.counters + k * kCounterStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
      a.counters[k * kCounterStride] = 0u;
  }
  if (!a.update) return;
  const float mean = block_mean_of(msum, N);
  for (int n = threadIdx.x; n < N; n += kBlock) {
    const float2 v = vs[n];
    const float mag = mag32(v);
    SpotRec r = a.recs ? a.recs[n] : a.sp[n];
    if (!update_rec(r, v, mag, mean)) {
      a.status[0] = 4;  // HG_ENUMERIC
      if (a.recs && !a.chain) a.sp[n] = r;  // the state this pass used
      continue;
    }
    if (a.chain) store_rec_dev(a.sp + n, r);
    else a.sp[n] = r;
    // C_n = A_n e^{i theta_n} = A_n V_n / |V_n|
    const float Am = r.A / mag;
    if (a.chain) store_dev(a.coef + n, make_float2(Am * v.x, Am * v.y));
    else a.coef[n] = make_float2(Am * v.x, Am * v.y);
  }
}

// Pending pass: every block adds the rows of the previous pass's total set
// (integer sums: the total that a hand-off would have formed), applies that
// pass's update to the state before it and keeps the result in recs (LDS),
// with the arithmetic and the mean of tail_final; with cl, also
// C_n = A_n e^{i theta_n} in FP32 (LDS), formed as tail_final forms it.
// Block 0 (lead) also clears the total set two passes back, stores the state
// for the next pass when this pass defers in turn (the final state, in the
// final hologram), the previous V when traced, and the status. 
//
// load() only requests the values, so that what the caller does before
// apply() overlaps their way.  The totals were completed by the launch before
// this one: ordinary 16-byte loads read them, which the blocks of an XCD
// share in its L2 (device-scope loads of 8 bytes, each a trip to memory,
// took 0.65 us more per compressed pass of 1296 blocks at N = 100).
typedef unsigned long long ull2_t __attribute__((ext_vector_type(2)));
typedef float flt4_t __attribute__((ext_vector_type(4)));
template <int MAXN>
struct PendingState {
  static constexpr int kPer = (MAXN + kBlock - 1) / kBlock;
  static_assert(sizeof(SpotRec) == 2 * sizeof(flt4_t), "a record is two 16-byte words");
  ull2_t sum[kPer];  // modulo 2^64: the exact total fits
  flt4_t lo[kPer], hi[kPer];

  // st: the state before the update; tot: the total set's first row.
  __device__ __forceinline__ void load(const SpotRec* st, const unsigned long long* tot, int N) {
    if (MAXN < kAccWideSpots || N < kAccWideSpots) load_rows<kAccRows>(st, tot, N);
    else load_rows<kAccRowsWide>(st, tot, N);
  }
  template <int ROWS>
  __device__ __forceinline__ void load_rows(const SpotRec* st, const unsigned long long* tot,
                                            int N) {
    const int stride = acc_row_words(N) / kAccSpotWords;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int n = threadIdx.x + i * kBlock;
      sum[i] = ull2_t{0ull, 0ull};
      lo[i] = hi[i] = flt4_t{0.f, 0.f, 0.f, 0.f};
      if (n < N) {
        const HG_GLOBAL ull2_t* q = as_global(reinterpret_cast<const ull2_t*>(tot)) + n;
        ull2_t v[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) v[r] = q[r * stride];
        const HG_GLOBAL flt4_t* s = as_global(reinterpret_cast<const flt4_t*>(st + n));
        lo[i] = s[0];
        hi[i] = s[1];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) sum[i] += v[r];
      }
    }
  }

  // D: PassDesc, SepDesc or MxDesc.  Every thread calls it (block barriers).
  template <typename D>
  __device__ __forceinline__ void apply(const JobDev& jb, const D& d, int N, bool lead,
                                        SpotRec* recs, float2* cl) const {
    double2 t[kPer];
    float msum = 0.f;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      t[i] = make_double2((double)(long long)sum[i][0] * d.prev_inv,
                          (double)(long long)sum[i][1] * d.prev_inv);
      if ((int)threadIdx.x + i * kBlock < N) msum += mag32(field32(t[i]));
    }
    const float mean = block_mean_of(msum, N);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int n = threadIdx.x + i * kBlock;
      if (n >= N) continue;
      SpotRec r;
      r.cx = lo[i][0];
      r.cy = lo[i][1];
      r.cz = lo[i][2];
      r.th = lo[i][3];
      r.A = hi[i][0];
      r.a0 = hi[i][1];
      r.w = hi[i][2];
      r.pad = hi[i][3];
      const float2 v = field32(t[i]);
      const float mag = mag32(v);
      const bool ok = update_rec(r, v, mag, mean);
      if (!ok && lead) jb.status[0] = 4;  // HG_ENUMERIC
      if (cl) {  // C_n = A_n e^{i theta_n}
        float2 C;
        if (ok) {
          const float Am = r.A / mag;  // as tail_final forms it
          C = make_float2(Am * v.x, Am * v.y);
        } else {
          float sn, cs;
          sincos_turns(r.th, sn, cs);
          C = make_float2(r.A * cs, r.A * sn);
        }
        cl[n] = C;
      }
      const flt4_t a = {r.cx, r.cy, r.cz, r.th}, b = {r.A, r.a0, r.w, r.pad};
      flt4_t* dst = reinterpret_cast<flt4_t*>(recs + n);
      dst[0] = a;
      dst[1] = b;
      if (lead && d.st_out) {
        HG_GLOBAL flt4_t* out = as_global_mut(reinterpret_cast<flt4_t*>(d.st_out + n));
        out[0] = a;
        out[1] = b;
      }
      if (lead && d.prev_V) {
        HG_GLOBAL double* q = as_global_mut(reinterpret_cast<double*>(d.prev_V + n));
        q[0] = t[i].x;
        q[1] = t[i].y;
      }
    }
    __syncthreads();
    if (lead && d.clear_row >= 0) {
      HG_GLOBAL unsigned long long* q =
          as_global_mut(jb.acc + d.clear_row * acc_set_words(N));
      for (int k = threadIdx.x; k < acc_set_words(N); k += kBlock)
        __hip_atomic_store(q + k, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};
template <int MAXN, typename D>
__device__ __forceinline__ void apply_pending(const JobDev& jb, const D& d, bool lead,
                                              SpotRec* recs, float2* cl) {
  PendingState<MAXN> ps;
  ps.load(d.st_in, jb.acc + d.prev_row * acc_set_words(jb.N), jb.N);
  ps.apply(jb, d, jb.N, lead, recs, cl);
}

// Chained launch: the update of this pass is complete (this block's state
// stores first), so the next pass may start.
__device__ void publish_gen(const PassCtx& a) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if ((int)threadIdx.x < kGenCopies)
    __hip_atomic_store(a.gen + threadIdx.x * kCounterStride, a.gen_next, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// Counts `count` tiles listed in done[] into their groups (the block's own
// additions to the group sums are complete first); the groups this block
// completes are appended to owned[].
constexpr int kDoneList = 256;  // = kBlock: one counting thread per tile
constexpr int kMaxGroups = 128;
__device__ void count_tiles(const PassCtx& a, const int* done, int count, int* owned,
                            int* nowned) {
  __builtin_amdgcn_s_waitcnt(0);  // this thread's atomic additions are complete
  __syncthreads();
  if ((int)threadIdx.x < count) {
    const int g = done[threadIdx.x] / a.plan.group_size;
    const int size = min(a.plan.group_size, a.plan.tiles - g * a.plan.group_size);
    if (atomicAdd(&a.counters[g * kCounterStride], 1u) == (unsigned)size - 1u) owned[atomicAdd(nowned, 1)] = g;
  }
  __syncthreads();
}

}  // namespace
}  // namespace hg
