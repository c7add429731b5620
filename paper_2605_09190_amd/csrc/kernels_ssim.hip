// kernels_ssim.hip - SSIM of two planes (Section 3's quality measure).
//
// SSIM = (2 mu_x mu_y + C1)(2 s_xy + C2) / ((mu_x^2 + mu_y^2 + C1)(s_x^2 + s_y^2 + C2)),
// C1 = (0.01 L)^2, C2 = (0.03 L)^2.
//   global : moments of the whole planes (population); the kernel returns the
//            five plane sums per workgroup, the host finishes the formula.
//   window7: the formula on every 7 x 7 window inside the plane (uniform
//            weights, sample moments), averaged over the windows.  A wave
//            takes 64 columns and walks down the rows: a row of both planes
//            through LDS, the five sums over seven neighbours of the row in
//            registers, the last seven rows' sums added up per window (105
//            operations a window before the formula, 245 when every window
//            summed its own 49 pixels, and 14 LDS reads instead of 98).
// Both write one FP64 partial per workgroup; the host adds them in a fixed
// order, so the result is reproducible.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

constexpr int kCols = 64, kWin = 7, kHalo = kWin - 1;

__device__ inline double load(const void* p, int dtype, int64_t stride, int y, int x) {
  const int64_t i = (int64_t)y * stride + x;
  return dtype == AQMP_F64 ? ((const double*)p)[i] : (double)((const float*)p)[i];
}

__device__ inline double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// A wave's rows come in `groups` of seven (the sums' places in the registers
// are then fixed): 7 groups - 6 rows of windows each.
// What bounds it: the FP64 instructions, once the loads are seven rows ahead
// (one row ahead: 43 us).  2048 x 1536 FP32: 26 us, 48 us with a 38 x 38 tile
// in LDS and 49 pixels summed per window.
template <typename T>
__global__ __launch_bounds__(256, 3) void k_ssim_window(const T* __restrict__ a, int64_t sa, const T* __restrict__ b,
                                                     int64_t sb, int w, int h, int groups, double c1, double c2,
                                                     double* __restrict__ partial) {
  __shared__ double sx[4][kCols + 8], sy[4][kCols + 8];
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int ow = w - kHalo, oh = h - kHalo;   // windows per row / column
  const int rows = kWin * groups - kHalo;
  const int tx0 = blockIdx.x * kCols, ty0 = (blockIdx.y * 4 + wv) * rows;
  const double n = kWin * kWin, inv_n = 1.0 / n, inv_n1 = 1.0 / (n - 1.0);
  double acc = 0.0;
  if (ty0 < oh) {
    const bool col = tx0 + lane < w, more = lane < kHalo && tx0 + kCols + lane < w, out = tx0 + lane < ow;
    // the next seven rows: the lane's column, and the six past the wave's
    T na[kWin], nb[kWin], ma[kWin], mb[kWin];
    auto fetch = [&](int r, int y) {
      const bool in = y < h;
      const T* ra = a + (int64_t)(in ? y : 0) * sa + tx0 + lane;
      const T* rb = b + (int64_t)(in ? y : 0) * sb + tx0 + lane;
      na[r] = in && col ? ra[0] : (T)0;
      nb[r] = in && col ? rb[0] : (T)0;
      ma[r] = in && more ? ra[kCols] : (T)0;
      mb[r] = in && more ? rb[kCols] : (T)0;
    };
    double s[kWin][5];
#pragma unroll
    for (int r = 0; r < kWin; ++r)
#pragma unroll
      for (int k = 0; k < 5; ++k) s[r][k] = 0.0;
#pragma unroll
    for (int r = 0; r < kWin; ++r) fetch(r, ty0 + r);
    for (int g = 0; g < groups; ++g)
#pragma unroll
      for (int r = 0; r < kWin; ++r) {
        const int i = kWin * g + r;            // row ty0 + i
        sx[wv][lane] = (double)na[r];
        sy[wv][lane] = (double)nb[r];
        if (lane < kHalo) {
          sx[wv][kCols + lane] = (double)ma[r];
          sy[wv][kCols + lane] = (double)mb[r];
        }
        if (g + 1 < groups) fetch(r, ty0 + i + kWin);
        wave_sync();
        double q[5] = {0, 0, 0, 0, 0};
#pragma unroll
        for (int d = 0; d < kWin; ++d) {
          const double u = sx[wv][lane + d], v = sy[wv][lane + d];
          q[0] += u;
          q[1] += v;
          q[2] = fma(u, u, q[2]);
          q[3] = fma(v, v, q[3]);
          q[4] = fma(u, v, q[4]);
        }
        wave_sync();                           // read before the next row is written
#pragma unroll
        for (int k = 0; k < 5; ++k) s[r][k] = q[k];
        if (i >= kHalo && ty0 + i - kHalo < oh) {
          double m[5];
#pragma unroll
          for (int k = 0; k < 5; ++k)
            m[k] = ((s[0][k] + s[1][k]) + (s[2][k] + s[3][k])) + ((s[4][k] + s[5][k]) + s[6][k]);
          const double mx = m[0] * inv_n, my = m[1] * inv_n;
          const double vx = (m[2] - m[0] * mx) * inv_n1, vy = (m[3] - m[1] * my) * inv_n1;
          const double cxy = (m[4] - m[0] * my) * inv_n1;
          const double v = ((2 * mx * my + c1) * (2 * cxy + c2)) / ((mx * mx + my * my + c1) * (vx + vy + c2));
          acc += out ? v : 0.0;
        }
      }
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) partial[blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

__global__ __launch_bounds__(256) void k_ssim_moments(const void* a, int64_t sa, const void* b, int64_t sb, int dtype,
                                                      int w, int h, double* partial) {
  __shared__ double red[4];
  double s[5] = {0, 0, 0, 0, 0};
  const int64_t total = (int64_t)w * h;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int y = (int)(i / w), x = (int)(i % w);
    const double u = load(a, dtype, sa, y, x), v = load(b, dtype, sb, y, x);
    s[0] += u;
    s[1] += v;
    s[2] = fma(u, u, s[2]);
    s[3] = fma(v, v, s[3]);
    s[4] = fma(u, v, s[4]);
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const double r = block_sum(s[k], red);
    if (threadIdx.x == 0) partial[(size_t)blockIdx.x * 5 + k] = r;
  }
}

// Workgroups of 64 columns and four waves of 7 groups - 6 rows: the most
// groups (the fewest rows summed twice) that leave two waves per SIMD of the
// chip, at least two.  (2048 x 1536: three groups 26 us, four 29.)
struct SsimGrid {
  int x, y, groups;
};
SsimGrid ssim_grid(int w, int h) {
  SsimGrid g;
  g.x = (w - kHalo + kCols - 1) / kCols;
  for (g.groups = 4;; --g.groups) {
    const int per = 4 * (kWin * g.groups - kHalo);
    g.y = (h - kHalo + per - 1) / per;
    if (g.groups == 2 || (int64_t)g.x * g.y * 4 >= 2048) return g;
  }
}

}  // namespace

hipError_t launch_ssim(const aqmp_image& x, const aqmp_image& y, int mode, double c1, double c2, double* partial,
                       int* n_partial, hipStream_t s) {
  if (mode == AQMP_SSIM_WINDOW7) {
    const SsimGrid g = ssim_grid(x.w, x.h);
    const dim3 grid(g.x, g.y);
    *n_partial = (int)(grid.x * grid.y);
    if (x.dtype == AQMP_F64)
      hipLaunchKernelGGL(k_ssim_window<double>, grid, dim3(256), 0, s, (const double*)x.dev_ptr, x.row_stride,
                         (const double*)y.dev_ptr, y.row_stride, x.w, x.h, g.groups, c1, c2, partial);
    else
      hipLaunchKernelGGL(k_ssim_window<float>, grid, dim3(256), 0, s, (const float*)x.dev_ptr, x.row_stride,
                         (const float*)y.dev_ptr, y.row_stride, x.w, x.h, g.groups, c1, c2, partial);
  } else {
    *n_partial = kSsimMomentBlocks;
    hipLaunchKernelGGL(k_ssim_moments, dim3(kSsimMomentBlocks), dim3(256), 0, s, x.dev_ptr, x.row_stride,
                       y.dev_ptr, y.row_stride, x.dtype, x.w, x.h, partial);
  }
  return hipGetLastError();
}

}  // namespace aqmp

// ---------------------------------------------------------------------------
// Host entry: validates, launches, and finishes the mean on the host.
// ---------------------------------------------------------------------------
#include "host_util.h"

namespace aqmp {

int ssim_planes(const aqmp_image* x, const aqmp_image* y, int mode, double data_range, double* out, hipStream_t s) {
  if (!x || !y || !out) AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: null argument");
  if (!x->dev_ptr || !y->dev_ptr) AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: plane without data");
  if (x->w != y->w || x->h != y->h || x->dtype != y->dtype)
    AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: the planes need one size and one dtype");
  if (x->dtype != AQMP_F32 && x->dtype != AQMP_F64) AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: bad dtype");
  if (x->row_stride < x->w || y->row_stride < y->w) AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: row stride too small");
  if (mode != AQMP_SSIM_GLOBAL && mode != AQMP_SSIM_WINDOW7) AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: bad mode");
  if (mode == AQMP_SSIM_WINDOW7 ? (x->w < 7 || x->h < 7) : (x->w < 1 || x->h < 1))
    AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: plane too small for the mode");
  if (!(data_range > 0.0) || !std::isfinite(data_range)) AQMP_FAIL(AQMP_E_INVALID, "aqmp_ssim: bad data_range");
  const double c1 = (0.01 * data_range) * (0.01 * data_range), c2 = (0.03 * data_range) * (0.03 * data_range);
  const size_t cap = mode == AQMP_SSIM_WINDOW7
                         ? (size_t)ssim_grid(x->w, x->h).x * (size_t)ssim_grid(x->w, x->h).y
                         : (size_t)kSsimMomentBlocks * 5;
  double* d_part = nullptr;
  int rc = dev_alloc((void**)&d_part, cap * sizeof(double));
  if (rc != AQMP_OK) return rc;
  int np = 0;
  hipError_t e = launch_ssim(*x, *y, mode, c1, c2, d_part, &np, s);
  std::vector<double> h(mode == AQMP_SSIM_WINDOW7 ? (size_t)np : (size_t)np * 5);
  if (e == hipSuccess) e = hipMemcpyAsync(h.data(), d_part, h.size() * sizeof(double), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  dev_free(d_part, cap * sizeof(double));
  if (e != hipSuccess) AQMP_FAIL(AQMP_E_HIP, std::string("aqmp_ssim: ") + hipGetErrorString(e));
  if (mode == AQMP_SSIM_WINDOW7) {
    double sum = 0.0;
    for (double v : h) sum += v;
    *out = sum / ((double)(x->w - 6) * (double)(x->h - 6));
  } else {
    double m[5] = {0, 0, 0, 0, 0};
    for (int b = 0; b < np; ++b)
      for (int k = 0; k < 5; ++k) m[k] += h[(size_t)b * 5 + k];
    const double n = (double)x->w * (double)x->h;
    const double mx = m[0] / n, my = m[1] / n;
    const double vx = m[2] / n - mx * mx, vy = m[3] / n - my * my, cxy = m[4] / n - mx * my;
    *out = ((2 * mx * my + c1) * (2 * cxy + c2)) / ((mx * mx + my * my + c1) * (vx + vy + c2));
  }
  return AQMP_OK;
}

}  // namespace aqmp
