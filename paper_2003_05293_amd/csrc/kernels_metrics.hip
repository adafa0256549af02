// FP64 metrics of a hologram (paper section 2, last paragraph, and eq. 7):
// the spot fields V*_n = mean over the pupil of A(p) e^{i (Phi(p) - phi_n(p))}.
//
// eq. (2) splits into a part in x' and a part in y', so e^{-i phi_n(i,j)} =
// Ex[i][n] Ey[j][n] and V*_n = sum_j Ey[j][n] T[j][n] / |Omega| with
// T = U Ex, U(j, i) = A e^{i Phi}: a complex matrix product, run on the FP64
// matrix cores.
#include <math.h>

#include "device_common.hpp"
#include "kernels.hpp"

namespace hg {

namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4_t mfma64(double a, double b, const d4_t& c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Ex [Wp][Np] and Ey [Hp][Np] (kernels.hpp), zero beyond the grid and N.
__global__ void k_metric_tables(SetupArgs a, SpotPtrs in, double2* __restrict__ Ex,
                                double2* __restrict__ Ey) {
  const int Np = metric_spots(a.N), Wp = metric_cols(a.W), Hp = metric_rows(a.H);
  const int64_t nx = (int64_t)Wp * Np, ny = (int64_t)Hp * Np;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nx + ny) return;
  const bool is_x = k < nx;
  const int64_t kk = is_x ? k : k - nx;
  const int pix = (int)(kk / Np);
  const int n = (int)(kk % Np);
  const int len = is_x ? a.W : a.H;
  double s = 0.0, c = 0.0;
  if (pix < len && n < a.N) {
    const double off = ((double)pix - 0.5 * (double)(len - 1)) * a.pitch_mm;
    const double lat = is_x ? in.x[n] : in.y[n];
    const double z = in.z[n];
    const double lf = a.lambda_mm * a.focal_mm;
    const double lf2 = lf * a.focal_mm;
    double t = lat * off / lf + z * off * off / lf2;  // turns
    t -= rint(t);
    sincospi(2.0 * t, &s, &c);
  }
  (is_x ? Ex : Ey)[kk] = make_double2(c, -s);
}

// One block: 64 rows (16 per wave) times the columns of its split, in chunks
// of at most kMetricCols.  Per chunk every lane forms u of its pixels once,
// in the order of the A operand (row l % 16, column 4 q + l / 16 of column
// quad q; wave-private LDS, no barrier), then for up to four 16-spot blocks
// at a time T = U Ex (two products each for re and im per quad; re and im
// are separate operands, so no pixel's sine is formed twice), the product
// with Ey, the sum over the rows, and the block's sums in `partial`.
//
// v_mfma_f64_16x16x4_f64: A[l % 16][l / 16], B[l / 16][l % 16],
// D[l / 16 + 4 r][l % 16] for lane l, r < 4.
//
// Bound: the FP64 matrix cores (8 W H Np operations, 16.5 us at 1152^2 and 112
// padded spots and the 72 TFLOP/s that a large product reaches) and, beside them, a
// sine and cosine per pixel.  At 1152^2, N = 100: 33 us, and 5 us for the
// reduction; one thread per spot over four rows, with every term's Ex from the
// L2, took 671 us and its reduction (one thread per spot) 69 us.  The whole
// call: 796 to 73 us.
constexpr int kMetricBlocks = 4;  // 16-spot blocks per pass over the chunk
template <int R>
__device__ __forceinline__ void metric_spots_pass(const double2* __restrict__ Ex,
                                                  const double2* __restrict__ Ey, int Np, int N,
                                                  const double2 (*us)[64], int quads, int c0,
                                                  int row0, int sb0, double2 (*red)[64],
                                                  double2* partial, bool add) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int wave = threadIdx.x >> 6;
  d4_t tr[R], ti[R];
#pragma unroll
  for (int k = 0; k < R; ++k) tr[k] = ti[k] = d4_t{0.0, 0.0, 0.0, 0.0};
  const double2* e0 = Ex + (int64_t)(c0 + lg) * Np + 16 * sb0 + lr;
  double2 e[R], f[R];
#pragma unroll
  for (int k = 0; k < R; ++k) e[k] = e0[16 * k];
  for (int q = 0; q < quads; ++q) {
    const double2 u = us[q][lane];
    const double2* en = e0 + (int64_t)4 * (q + 1 < quads ? q + 1 : q) * Np;
#pragma unroll
    for (int k = 0; k < R; ++k) f[k] = en[16 * k];  // the next quad's operands
    const double nui = -u.y;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      tr[k] = mfma64(u.x, e[k].x, tr[k]);
      ti[k] = mfma64(u.x, e[k].y, ti[k]);
      tr[k] = mfma64(nui, e[k].y, tr[k]);
      ti[k] = mfma64(u.y, e[k].x, ti[k]);
    }
#pragma unroll
    for (int k = 0; k < R; ++k) e[k] = f[k];
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    double vr = 0.0, vi = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double2 y = Ey[(int64_t)(row0 + lg + 4 * r) * Np + 16 * (sb0 + k) + lr];
      vr = fma(tr[k][r], y.x, fma(-ti[k][r], y.y, vr));
      vi = fma(tr[k][r], y.y, fma(ti[k][r], y.x, vi));
    }
    vr += __shfl_xor(vr, 16);
    vi += __shfl_xor(vi, 16);
    vr += __shfl_xor(vr, 32);
    vi += __shfl_xor(vi, 32);
    if (lg == 0) red[wave][16 * k + lr] = make_double2(vr, vi);
  }
  __syncthreads();
  const int n = 16 * sb0 + (int)threadIdx.x;
  if ((int)threadIdx.x < 16 * R && n < N) {
    double2 v = red[0][threadIdx.x];
    for (int w = 1; w < kWaves; ++w) {
      v.x += red[w][threadIdx.x].x;
      v.y += red[w][threadIdx.x].y;
    }
    if (add) {  // (this thread's own sum of the chunks before)
      v.x += partial[n].x;
      v.y += partial[n].y;
    }
    partial[n] = v;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kBlock, 2) void k_metric_tiles(
    const double2* __restrict__ Ex, const double2* __restrict__ Ey, int N, int W, int H, int cols,
    int chunk, const float* __restrict__ phi, int32_t ap_q, double ill_a,
    double2* __restrict__ partial) {
  extern __shared__ double2 metric_lds[];  // [kWaves][chunk / 4][64]
  __shared__ double2 red[kWaves][64];
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int wave = threadIdx.x >> 6;
  const int Np = metric_spots(N), S16 = Np / 16;
  const int row0 = (int)blockIdx.y * kMetricRows + 16 * wave, row = row0 + lr;
  double2(*us)[64] = reinterpret_cast<double2(*)[64]>(metric_lds + (size_t)wave * chunk * 16);
  double2* out = partial + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * N;
  const bool pupil = ap_q >= 0 || ill_a > 0.0;
  const int c1 = min(W, ((int)blockIdx.x + 1) * cols);
  bool add = false;
  for (int c0 = (int)blockIdx.x * cols; c0 < c1; c0 += chunk) {
    const int quads = (min(chunk, c1 - c0) + 3) / 4;
    for (int q = 0; q < quads; ++q) {
      const int col = c0 + 4 * q + lg;
      double2 u = make_double2(0.0, 0.0);
      if (row < H && col < c1) {
        double s, c;
        sincos((double)phi[(int64_t)row * W + col], &s, &c);
        if (pupil) {
          const int64_t lx = 2 * (int64_t)col - (W - 1), ly = 2 * (int64_t)row - (H - 1);
          const int64_t Q = lx * lx + ly * ly;
          const double wt =
              (ap_q >= 0 && Q > ap_q) ? 0.0 : (ill_a > 0.0 ? exp(-(double)Q * ill_a) : 1.0);
          c *= wt;
          s *= wt;
        }
        u = make_double2(c, s);
      }
      us[q][lane] = u;
    }
    int sb0 = 0;
    for (; sb0 + kMetricBlocks <= S16; sb0 += kMetricBlocks)
      metric_spots_pass<kMetricBlocks>(Ex, Ey, Np, N, us, quads, c0, row0, sb0, red, out, add);
    switch (S16 - sb0) {
      case 3: metric_spots_pass<3>(Ex, Ey, Np, N, us, quads, c0, row0, sb0, red, out, add); break;
      case 2: metric_spots_pass<2>(Ex, Ey, Np, N, us, quads, c0, row0, sb0, red, out, add); break;
      case 1: metric_spots_pass<1>(Ex, Ey, Np, N, us, quads, c0, row0, sb0, red, out, add); break;
      default: break;
    }
    add = true;
  }
}

// Sums of the blocks' partials in a fixed order: 16 spots per block, thread
// (spot, slice s of 16) adds the partials s, s + 16, ..., the slices are
// added in order.  V and the status word go straight to the caller's pinned
// host memory; the sticky status is cleared once reported.
__global__ __launch_bounds__(256) void k_metric_reduce(const double2* __restrict__ partial,
                                                       int nblk, int N, double inv_count,
                                                       double2* __restrict__ V, int32_t* status,
                                                       int32_t* __restrict__ status_out) {
  __shared__ double2 part[16][16];
  const int c = threadIdx.x & 15, s = threadIdx.x >> 4;
  const int n = blockIdx.x * 16 + c;
  double re = 0.0, im = 0.0;
  if (n < N) {
#pragma unroll 8
    for (int b = s; b < nblk; b += 16) {
      const double2 v = partial[(int64_t)b * N + n];
      re += v.x;
      im += v.y;
    }
  }
  part[s][c] = make_double2(re, im);
  __syncthreads();
  if (s == 0 && n < N) {
    for (int k = 1; k < 16; ++k) {
      re += part[k][c].x;
      im += part[k][c].y;
    }
    V[n] = make_double2(re * inv_count, im * inv_count);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int32_t st = *status;
    *status_out = st;
    if (st) *status = 0;
  }
}

}  // namespace

MetricPlan plan_metrics(int W, int H) {
  // about two blocks per compute unit; no split below 16 columns
  MetricPlan p;
  p.row_groups = metric_rows(H) / kMetricRows;
  int splits = 512 / p.row_groups;
  if (splits < 1) splits = 1;
  if (splits > ceil_div(W, 16)) splits = ceil_div(W, 16);
  p.cols = (ceil_div(W, splits) + 3) / 4 * 4;
  p.splits = ceil_div(W, p.cols);
  p.chunk = p.cols < kMetricCols ? p.cols : kMetricCols;
  return p;
}

void launch_metric_tables(const SetupArgs& a, const SpotPtrs& in, double2* Ex, double2* Ey,
                          hipStream_t s) {
  const int64_t total =
      (int64_t)(metric_cols(a.W) + metric_rows(a.H)) * metric_spots(a.N);
  hipLaunchKernelGGL(k_metric_tables, dim3(ceil_div(total, 256)), dim3(256), 0, s, a, in, Ex,
                     Ey);
}

void launch_metric_tiles(const MetricPlan& p, const double2* Ex, const double2* Ey, int N, int W,
                         int H, const float* phi, int32_t ap_q, double ill_a, double2* partial,
                         hipStream_t s) {
  const size_t shmem = sizeof(double2) * kWaves * 16 * (size_t)p.chunk;
  hipLaunchKernelGGL(k_metric_tiles, dim3(p.splits, p.row_groups), dim3(kBlock), shmem, s, Ex, Ey,
                     N, W, H, p.cols, p.chunk, phi, ap_q, ill_a, partial);
}

void launch_metric_reduce(const double2* partial, int nblk, int N, double inv_count,
                          double2* V_host, int32_t* status, int32_t* status_host, hipStream_t s) {
  hipLaunchKernelGGL(k_metric_reduce, dim3(ceil_div(N, 16)), dim3(256), 0, s, partial, nblk, N,
                     inv_count, V_host, status, status_host);
}

}  // namespace hg
