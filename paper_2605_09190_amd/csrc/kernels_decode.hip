// kernels_decode.hip - the decoder (Algorithm 3): every leaf of a job writes
// sum_t c_t phi_{i_t} at its position, all block sizes in one launch.
//
// A job's nodes are contiguous in every level (the split scan keeps the
// order of the jobs and writes each job's range, see k_split_emit), so a
// launch visits that job's nodes only.  Work is dealt out in tasks of one
// workgroup: one block of 64 (a 16-row strip per wave), four of 32 or 16 (one
// per wave), 16 of 8 or 64 of 4.  The lanes of a node load its records
// together and hand them round, and the table rows of four atoms are in
// flight at once.
//
// What bounds it: for one small plane the chain of cold loads (ranges, node,
// records, table) of a short kernel; for many nodes what the L1 returns per
// atom, 64 bytes per clock.  So blocks of 16 and more take 8 bytes of either
// table row per lane and atom instead of 32 (see decode_rows).  One plane of
// 2048 x 2048 (12 144 + 24 940 + 52 563 + 56 897 atom steps of 64, 32, 16 and
// 8), of 1024 x 768 in a search, of 1000 x 667 in FP64: 21.8, 11.9 and 10.5
// us; with rows of four pixels per lane 26.2, 14.9 and 12.4.  More atoms in
// flight (8: 22.7 / 12.4 us), fewer rows per lane (one: 36 / 17.8) and fewer
// registers for more waves (80: 21.5 / 13.2) are slower.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

typedef __attribute__((address_space(1))) const double dc_cf64;

template <int N>
struct DecGeo {
  static constexpr int K = N * N;
  static constexpr int LPN = N >= 16 ? 64 : N * N / 4;         // lanes of one node (N = 64: of one strip)
  static constexpr int NPT = N == 64 ? 1 : 4 * (64 / LPN);     // nodes per task
};

// acc[i] += w' x, w' lane i's w of the lane's row of 16: four rows at a time.
// (A value is read across lanes two wait states after it is written.)
template <int R>
__device__ inline void add_rows(double (&acc)[R], double w, double x) {
#define AQMP_ROWS4(I)                                                                                          \
  asm("s_nop 1\n\t"                                                                                            \
        "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"                             \
        "v_fmac_f64_dpp %1, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"                             \
        "v_fmac_f64_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"                             \
        "v_fmac_f64_dpp %3, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"                                 \
        : "+v"(acc[I]), "+v"(acc[I + 1]), "+v"(acc[I + 2]), "+v"(acc[I + 3])                                   \
        : "v"(w), "v"(x), "n"(I), "n"(I + 1), "n"(I + 2), "n"(I + 3));
  AQMP_ROWS4(0)
  if constexpr (R == 16) {
    AQMP_ROWS4(4)
    AQMP_ROWS4(8)
    AQMP_ROWS4(12)
  }
#undef AQMP_ROWS4
}

__device__ inline void put(void* out, int32_t dtype, int64_t at, double v) {
  if (dtype == AQMP_F64)
    ((double*)out)[at] = v;
  else
    ((float*)out)[at] = (float)v;
}

// N >= 16: a wave takes 16 rows of a block of 64, or a whole smaller block.  A
// lane holds one column of N and R rows of it, so that an atom costs two
// table loads of 8 bytes: T[q] at the lane's column and, for the R rows, R
// values of c T[p] spread over the lanes of its row of 16, from where each is
// broadcast by the multiply-add that takes it.
template <int N>
__device__ inline void decode_rows(const DecodeLevel& L, int first, int end, const JobDev* __restrict__ jobs, int job,
                                   double step, void* out, int32_t dtype, int64_t row_stride) {
  constexpr int K = N * N, U = 4;
  constexpr int R = N == 16 ? 4 : 16;                          // rows per lane
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int node = N == 64 ? first : first + wv;
  if (node >= end) return;
  const uint8_t st = L.lv.st[node];
  const int na = __builtin_amdgcn_readfirstlane(L.lv.t[node]);
  const int bx = L.lv.x0[node], by = L.lv.y0[node];
  const int w = jobs[job].w, h = jobs[job].h;
  const size_t rec = (size_t)node * L.lv.kmax;
  int ri = 0;
  double rc = 0.0;
  if (lane < L.lv.kmax) {   // loaded with the node's values; the first na are its atoms
    ri = L.lv.rec_idx[rec + lane];
    rc = L.lv.rec_coef[rec + lane];
  }
  if (st & ST_SPLIT) return;
  const int x = lane & (N - 1), y0 = (N == 64 ? 16 * wv : 0) + lane / N * R;
  const dc_cf64* tab = (const dc_cf64*)L.tab;
  const uint32_t ox = (uint32_t)x, oy = (uint32_t)(y0 + (lane & (R - 1)));
  double acc[R];
#pragma unroll
  for (int i = 0; i < R; ++i) acc[i] = 0.0;
  for (int base = 0; base < na; base += 64) {
    const int cnt = na - base < 64 ? na - base : 64;
    if (base > 0 && lane < cnt) {
      ri = L.lv.rec_idx[rec + base + lane];
      rc = L.lv.rec_coef[rec + base + lane];
    }
    if (step > 0.0) rc = rint(rc / step) * step;
    for (int s = 0; s < cnt; s += U) {
      double c[U], vx[U], vy[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = s + u < cnt ? s + u : cnt - 1;
        const int a = __builtin_amdgcn_readlane(ri, k);
        const unsigned long long cu = (unsigned long long)__double_as_longlong(rc);
        const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)cu, k);
        const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(cu >> 32), k);
        c[u] = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        const int f = a / K, q = (a % K) / N, pp = a % N;
        vx[u] = tab[(uint32_t)(f * K + q * N) + ox];
        vy[u] = tab[(uint32_t)(f * K + pp * N) + oy];
        if (a % K == 0) {   // the constant atom: 1 / N exactly
          vx[u] = 1.0 / N;
          vy[u] = 1.0;
        }
        vy[u] *= c[u];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u < cnt)
          add_rows<R>(acc, vy[u], vx[u]);
    }
  }
  // Pixels of the padding (past the image) are not written.
  if (bx + x >= w) return;
#pragma unroll
  for (int i = 0; i < R; ++i)
    if (by + y0 + i < h) put(out, dtype, (int64_t)(by + y0 + i) * row_stride + bx + x, acc[i]);
}

// N = 4 and 8: 4 and 16 lanes per node, a row of four pixels per lane.
template <int N>
__device__ inline void decode_small(const DecodeLevel& L, int first, int end, const JobDev* __restrict__ jobs, int job,
                                    double step, void* out, int32_t dtype, int64_t row_stride, bool wide) {
  using G = DecGeo<N>;
  constexpr int K = G::K, LPN = G::LPN, U = 4;
  const int lane = threadIdx.x & 63, li = lane % LPN;
  const int node = first + (int)threadIdx.x / LPN;
  const bool live = node < end && !(L.lv.st[node < end ? node : first] & ST_SPLIT);
  if (__ballot(live) == 0ull) return;
  const int nd = live ? node : first;
  const int na = live ? L.lv.t[nd] : 0;
  const int px = 4 * (li & (N / 4 - 1)), py = li / (N / 4);
  const int x = L.lv.x0[nd] + px, y = L.lv.y0[nd] + py;
  const dc_cf64* tab = (const dc_cf64*)L.tab;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  int nmax = na;   // the longest list of the wave's nodes
#pragma unroll
  for (int off = LPN; off < 64; off <<= 1) {
    const int o = __shfl_xor(nmax, off, 64);
    nmax = o > nmax ? o : nmax;
  }
  nmax = __builtin_amdgcn_readfirstlane(nmax);
  const size_t rec = (size_t)nd * L.lv.kmax;
  for (int base = 0; base < nmax; base += LPN) {
    const int mine = base + li;
    int ri = 0;
    double rc = 0.0;
    if (mine < na) {
      ri = L.lv.rec_idx[rec + mine];
      rc = L.lv.rec_coef[rec + mine];
      if (step > 0.0) rc = rint(rc / step) * step;
    }
    const int cnt = nmax - base < LPN ? nmax - base : LPN;
    for (int s = 0; s < cnt; s += U) {
      double c[U], tx[U][4], ty[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int src = (lane & ~(LPN - 1)) + (s + u < cnt ? s + u : cnt - 1);
        const int a = __shfl(ri, src, 64);
        c[u] = __shfl(rc, src, 64);
        const int f = a / K, q = (a % K) / N, p = a % N;
        const bool dc = a % K == 0;   // the constant atom: 1 / N exactly
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double v = tab[(uint32_t)(f * K + q * N + px) + j];
          tx[u][j] = dc ? 1.0 / N : v;
        }
        const double v = tab[(uint32_t)(f * K + p * N + py)];
        ty[u] = dc ? 1.0 : v;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (base + s + u < na)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = fma(c[u], ty[u] * tx[u][j], acc[j]);
    }
  }
  // Pixels of the padding (past the image) are not written.
  const int w = jobs[job].w;
  if (!live || y >= jobs[job].h) return;
  const int64_t at = (int64_t)y * row_stride + x;
  if (wide && x + 3 < w) {
    if (dtype == AQMP_F64) {
      *(double2*)((double*)out + at) = make_double2(acc[0], acc[1]);
      *(double2*)((double*)out + at + 2) = make_double2(acc[2], acc[3]);
    } else {
      *(float4*)((float*)out + at) = make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (x + j < w) put(out, dtype, at + j, acc[j]);
  }
}

__global__ __launch_bounds__(256) void k_decode(DecodeArgs a, double step, void* out, int32_t dtype,
                                                int64_t row_stride, int32_t wide) {
  // the job's nodes per level; a level below one without nodes has none (its
  // range may be left from an earlier encode)
  int b[kLevels], e[kLevels], task0[kLevels + 1];
  int n_tasks = 0;
  bool any = true;
  int2 rg[kLevels];   // all at once: a level not of the job's is read and not used
#pragma unroll
  for (int l = 2; l < kLevels; ++l) rg[l] = a.ranges[(size_t)l * a.n_jobs + a.job];
#pragma unroll
  for (int l = kLevels - 1; l >= 2; --l) {
    b[l] = e[l] = 0;
    task0[l] = n_tasks;
    if (l <= a.lg_hi && l >= a.lg_lo && any) {
      const int2 r = rg[l];
      b[l] = r.x;
      e[l] = r.y;
      any = r.y > r.x;
      constexpr int npt[kLevels] = {1, 1, DecGeo<4>::NPT, DecGeo<8>::NPT, DecGeo<16>::NPT, DecGeo<32>::NPT, DecGeo<64>::NPT};
      n_tasks += (r.y - r.x + npt[l] - 1) / npt[l];
    }
  }
  for (int t = blockIdx.x; t < n_tasks; t += gridDim.x) {
#define AQMP_DEC(LG, NN, FN, ...)                                                                                    \
  if (e[LG] > b[LG] && t >= task0[LG] && t - task0[LG] < (e[LG] - b[LG] + DecGeo<NN>::NPT - 1) / DecGeo<NN>::NPT) { \
    FN<NN>(a.lv[LG], b[LG] + (t - task0[LG]) * DecGeo<NN>::NPT, e[LG], a.jobs, a.job, step, out, dtype, __VA_ARGS__); \
    continue;                                                                                                        \
  }
    AQMP_DEC(6, 64, decode_rows, row_stride)
    AQMP_DEC(5, 32, decode_rows, row_stride)
    AQMP_DEC(4, 16, decode_rows, row_stride)
    AQMP_DEC(3, 8, decode_small, row_stride, wide != 0)
    AQMP_DEC(2, 4, decode_small, row_stride, wide != 0)
#undef AQMP_DEC
  }
}

}  // namespace

// blocks_px: pixels of the job's padded plane.  A workgroup per 1 024 pixels
// (a task of small blocks), at most as many as are resident at once; the
// others are taken in turn.
hipError_t launch_decode(const DecodeArgs& a, int64_t blocks_px, double step, void* out, int32_t dtype, int64_t row_stride,
                         hipStream_t s) {
  int64_t g = (blocks_px + 1023) / 1024;
  if (g > 2048) g = 2048;
  if (g < 1) g = 1;
  // rows of four samples start 16 bytes apart when the plane and its stride do
  const int wide = ((uintptr_t)out % 16 == 0 && (row_stride * (dtype == AQMP_F64 ? 8 : 4)) % 16 == 0) ? 1 : 0;
  hipLaunchKernelGGL(k_decode, dim3((unsigned)g), dim3(256), 0, s, a, step, out, dtype, row_stride, wide);
  return hipGetLastError();
}

}  // namespace aqmp
