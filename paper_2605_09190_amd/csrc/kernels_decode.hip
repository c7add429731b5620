// kernels_decode.hip - the decoder (Algorithm 3): every leaf of a job writes
// sum_t c_t phi_{i_t} at its position, all block sizes in one launch.
//
// A job's nodes are contiguous in every level (the split scan keeps the
// order of the jobs and writes each job's range, see SplitOp), so a launch
// visits that job's nodes only.  Work is dealt out in tasks of one workgroup:
// one block of 64 (a 16-row strip per wave), four of 32 or 16 (one per wave),
// 16 of 8 or 64 of 4.  A lane holds rows of four pixels, so that a wave stores
// whole lines; the lanes of a node load its records together and hand them
// round, and the table rows of several atoms are in flight at once.
//
// What bounds it: the chain of a node's atoms (two dependent loads per batch
// of atoms), then the stores.  Three 2048 x 2048 planes: see launch_decode.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

typedef __attribute__((address_space(1))) const double dc_cf64;

template <int N>
struct DecGeo {
  static constexpr int K = N * N;
  static constexpr int LPN = N >= 16 ? 64 : N * N / 4;         // lanes of one node (N = 64: of one strip)
  static constexpr int RW = N >= 32 ? 4 : 1;                   // rows of four pixels per lane
  static constexpr int U = N >= 32 ? 2 : 4;                    // atoms whose table rows are in flight
  static constexpr int NPT = N == 64 ? 1 : 4 * (64 / LPN);     // nodes per task
  __device__ static int x(int li) { return N == 64 ? 4 * (li & 15) : 4 * (li & (N / 4 - 1)); }
  __device__ static int y(int li, int wv, int i) {
    if constexpr (N == 64) return 16 * wv + (li >> 4) + 4 * i;
    else if constexpr (N == 32) return (li >> 3) + 8 * i;
    else return li / (N / 4);
  }
};

template <int N>
__device__ inline void decode_task(const DecodeLevel& L, int first, int end, const JobDev* __restrict__ jobs, int job,
                                   double step, void* out, int dtype, int64_t row_stride, bool wide) {
  using G = DecGeo<N>;
  constexpr int K = G::K, LPN = G::LPN, RW = G::RW, U = G::U;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane % LPN;
  const double inv_n = 1.0 / N;
  int node = first + (N == 64 ? 0 : wv * (64 / LPN) + lane / LPN);
  if constexpr (LPN == 64) node = __builtin_amdgcn_readfirstlane(node);
  const bool live = node < end && !(L.lv.st[node < end ? node : first] & ST_SPLIT);
  if (__ballot(live) == 0ull) return;
  const int nd = live ? node : first;
  const int na = live ? L.lv.t[nd] : 0;
  const int bx = L.lv.x0[nd], by = L.lv.y0[nd];
  const dc_cf64* tab = (const dc_cf64*)L.tab;
  const int px = G::x(li);
  double acc[RW][4];
#pragma unroll
  for (int i = 0; i < RW; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
  // the longest list of the wave's nodes
  int nmax = na;
  if constexpr (LPN < 64) {
#pragma unroll
    for (int off = LPN; off < 64; off <<= 1) {
      const int o = __shfl_xor(nmax, off, 64);
      nmax = o > nmax ? o : nmax;
    }
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
      double c[U], tx[U][4], ty[U][RW];
      bool dc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = s + u < cnt ? s + u : cnt - 1;
        int a;
        if constexpr (LPN == 64) {
          a = __builtin_amdgcn_readlane(ri, k);
          const unsigned long long cu = (unsigned long long)__double_as_longlong(rc);
          const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)cu, k);
          const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(cu >> 32), k);
          c[u] = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        } else {
          const int src = (lane & ~(LPN - 1)) + k;
          a = __shfl(ri, src, 64);
          c[u] = __shfl(rc, src, 64);
        }
        const int f = a / K, q = (a % K) / N, p = a % N;
        dc[u] = p == 0 && q == 0;
        const dc_cf64* tf = tab + f * K;
#pragma unroll
        for (int j = 0; j < 4; ++j) tx[u][j] = tf[q * N + px + j];
#pragma unroll
        for (int i = 0; i < RW; ++i) ty[u][i] = tf[p * N + G::y(li, wv, i)];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (base + s + u < na) {
#pragma unroll
          for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const double phi = dc[u] ? inv_n : ty[u][i] * tx[u][j];
              acc[i][j] = fma(c[u], phi, acc[i][j]);
            }
        }
      }
    }
  }
  if (!live) return;
  // Pixels of the padding (past the image) are not written.
  const int w = jobs[job].w, h = jobs[job].h;
  const int x = bx + px;
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int y = by + G::y(li, wv, i);
    if (y >= h) continue;
    const int64_t at = (int64_t)y * row_stride + x;
    if (wide && x + 3 < w) {
      if (dtype == AQMP_F64) {
        *(double2*)((double*)out + at) = make_double2(acc[i][0], acc[i][1]);
        *(double2*)((double*)out + at + 2) = make_double2(acc[i][2], acc[i][3]);
      } else {
        *(float4*)((float*)out + at) =
            make_float4((float)acc[i][0], (float)acc[i][1], (float)acc[i][2], (float)acc[i][3]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (x + j >= w) continue;
        if (dtype == AQMP_F64)
          ((double*)out)[at + j] = acc[i][j];
        else
          ((float*)out)[at + j] = (float)acc[i][j];
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_decode(DecodeArgs a, double step, void* out, int32_t dtype,
                                                int64_t row_stride, int32_t wide) {
  // the job's nodes per level; a level below one without nodes has none (its
  // range may be left from an earlier encode)
  int b[kLevels], e[kLevels], task0[kLevels + 1];
  int n_tasks = 0;
  bool any = true;
#pragma unroll
  for (int l = kLevels - 1; l >= 2; --l) {
    b[l] = e[l] = 0;
    task0[l] = n_tasks;
    if (l <= a.lg_hi && l >= a.lg_lo && any) {
      const int2 r = a.ranges[(size_t)l * a.n_jobs + a.job];
      b[l] = r.x;
      e[l] = r.y;
      any = r.y > r.x;
      constexpr int npt[kLevels] = {1, 1, DecGeo<4>::NPT, DecGeo<8>::NPT, DecGeo<16>::NPT, DecGeo<32>::NPT, DecGeo<64>::NPT};
      n_tasks += (r.y - r.x + npt[l] - 1) / npt[l];
    }
  }
  for (int t = blockIdx.x; t < n_tasks; t += gridDim.x) {
#define AQMP_DEC(LG, NN)                                                                                             \
  if (e[LG] > b[LG] && t >= task0[LG] && t - task0[LG] < (e[LG] - b[LG] + DecGeo<NN>::NPT - 1) / DecGeo<NN>::NPT) { \
    decode_task<NN>(a.lv[LG], b[LG] + (t - task0[LG]) * DecGeo<NN>::NPT, e[LG], a.jobs, a.job, step, out, dtype,     \
                    row_stride, wide != 0);                                                                          \
    continue;                                                                                                        \
  }
    AQMP_DEC(6, 64)
    AQMP_DEC(5, 32)
    AQMP_DEC(4, 16)
    AQMP_DEC(3, 8)
    AQMP_DEC(2, 4)
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
