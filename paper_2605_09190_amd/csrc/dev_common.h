// dev_common.h - device helpers shared by the AQMP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aqmp {

// Round-to-nearest-even float -> bfloat16 bits (finite inputs).
__device__ __host__ inline uint16_t f32_to_bf16(float f) {
  uint32_t u;
  __builtin_memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Threads that cooperate on one quadtree node of size N: TPN threads per
// node (at most one 256-thread workgroup), NPW nodes per workgroup, PPT
// pixels per thread arranged as a PH x PW patch of the N x N block.
template <int N>
struct Geo {
  static constexpr int K = N * N;
  static constexpr int TPN = K < 256 ? K : 256;
  static constexpr int NPW = 256 / TPN;
  static constexpr int PPT = K / TPN;
  static constexpr int PH = PPT == 16 ? 4 : (PPT == 4 ? 2 : 1);
  static constexpr int PW = PPT / PH;
  static constexpr int PX = N / PW;   // patches per patch row
};

// Sum of v over the TPN threads of a node group, returned to every thread
// of the group.  Fixed butterfly order, then (TPN = 256) a fixed-order sum of
// the four wave totals: the result is bit-reproducible.  `scratch` must hold
// 4 doubles per group and the call must be reached by the whole workgroup.
template <int TPN>
__device__ inline double group_sum(double v, double* scratch) {
  constexpr int W = TPN < 64 ? TPN : 64;
#pragma unroll
  for (int off = 1; off < W; off <<= 1) v += __shfl_xor(v, off, 64);
  if constexpr (TPN > 64) {
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) scratch[w] = v;
    __syncthreads();
    v = (scratch[0] + scratch[1]) + (scratch[2] + scratch[3]);
  }
  return v;
}

// ---------------------------------------------------------------------------
// Decoupled look-back for stable single-pass prefix sums.  A tile word holds a
// flag in its top two bits (1: tile aggregate published, 2: inclusive prefix
// published) and a 32-bit count.  Tiles are taken in ticket order, so a tile
// only waits on tiles held by workgroups that started before it.  Each wait
// is bounded; when the bound runs out *err is set and the (then wrong) sum is
// used, so every wave still finishes.
// ---------------------------------------------------------------------------
constexpr unsigned long long kFlagAgg = 1ull << 62;
constexpr unsigned long long kFlagInc = 2ull << 62;
constexpr int kSpinLimit = 1 << 24;

__device__ inline unsigned long long load_acq(unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_rel(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-parallel look-back, called by all 64 lanes of one wave: publishes
// tile `tile`'s aggregate, then reads up to 64 predecessors per probe (lane i
// reads tile - 1 - i), stops at the nearest inclusive prefix, and publishes its
// own inclusive prefix.  Returns the exclusive prefix in every lane.
__device__ inline int lookback_wave(unsigned long long* tiles, int tile, int agg, int32_t* err) {
  const int lane = threadIdx.x & 63;
  if (tile == 0) {
    if (lane == 0) store_rel(&tiles[0], kFlagInc | (unsigned)agg);
    return 0;
  }
  if (lane == 0) store_rel(&tiles[tile], kFlagAgg | (unsigned)agg);
  int prefix = 0, end = tile, spins = 0;
  for (;;) {
    const int idx = end - 1 - lane;
    const unsigned long long v = idx >= 0 ? load_acq(&tiles[idx]) : (kFlagInc | 0ull);
    const unsigned fl = (unsigned)(v >> 62);
    const int val = (int)(unsigned)(v & 0xFFFFFFFFull);
    const unsigned long long inc = __ballot(fl == 2);
    const unsigned long long miss = __ballot(fl == 0);
    const unsigned long long upto = inc ? (inc & (~inc + 1ull)) : 0ull;   // lowest inclusive lane
    const unsigned long long need = inc ? (upto | (upto - 1ull)) : ~0ull;   // lanes that must be ready
    if (miss & need) {
      if (++spins > kSpinLimit) {
        if (lane == 0) atomicExch(err, 1);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    int x = ((need >> lane) & 1ull) ? val : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) x += __shfl_xor(x, off, 64);
    prefix += x;
    if (inc) break;
    end -= 64;
    spins = 0;
  }
  if (lane == 0) store_rel(&tiles[tile], kFlagInc | (unsigned)(prefix + agg));
  return prefix;
}

// Whole-wave reductions with DPP row operations (quad swaps, row mirrors,
// row broadcasts 15 and 31), then a read of lane 63: a fixed order, so the
// results are bit-reproducible, and no LDS-crossbar round trips.
template <int CTRL, int RM>
__device__ inline unsigned long long dpp_u64(unsigned long long v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, RM, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, RM, 0xF, false);
  return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}
__device__ inline unsigned long long lane63_u64(unsigned long long v) {
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)v, 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ inline unsigned long long wave_max_u64(unsigned long long v) {
#define AQMP_MAXSTEP(C, RM) { const unsigned long long o = dpp_u64<C, RM>(v); v = o > v ? o : v; }
  AQMP_MAXSTEP(0xB1, 0xF) AQMP_MAXSTEP(0x4E, 0xF) AQMP_MAXSTEP(0x141, 0xF)
  AQMP_MAXSTEP(0x140, 0xF) AQMP_MAXSTEP(0x142, 0xA) AQMP_MAXSTEP(0x143, 0xC)
#undef AQMP_MAXSTEP
  return lane63_u64(v);
}
// Orders the LDS writes of a wave's lanes before its later LDS reads by
// other lanes of the same wave (no workgroup barrier): the wave's LDS
// operations complete before it goes on (its loads and stores of global
// memory need not: none of them is read by another lane).
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Lane exchange with a permutation inside rows of 16 (every lane has a
// source, so there is no old value to keep), and lanes l and l ^ 16 or l ^ 32
// by a swap of a register against its copy (p the lower lane's value, q the
// upper's, in both lanes).  All VALU, no LDS round trip.
template <int CTRL>
__device__ inline uint32_t row_perm_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ inline double row_perm_f64(double d) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  const uint32_t lo = row_perm_u32<CTRL>((uint32_t)u), hi = row_perm_u32<CTRL>((uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int X>
__device__ inline void lane_pair_u32(uint32_t v, uint32_t& p, uint32_t& q) {
  static_assert(X == 16 || X == 32, "rows or halves");
  if constexpr (X == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    p = r[0];
    q = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    p = r[0];
    q = r[1];
  }
}
template <int X>
__device__ inline double lane_pair_sum_f64(double d) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  uint32_t p0, q0, p1, q1;
  lane_pair_u32<X>((uint32_t)u, p0, q0);
  lane_pair_u32<X>((uint32_t)(u >> 32), p1, q1);
  return __longlong_as_double((long long)(((unsigned long long)p1 << 32) | p0)) +
         __longlong_as_double((long long)(((unsigned long long)q1 << 32) | q0));
}

// Sum over the wave, the same bits in every lane: quads, eights, rows of 16,
// pairs of rows, halves.  (Row broadcasts into lane 63 add the same pairs,
// but need a zeroed register per exchange: 41 instructions instead of 24.)
__device__ inline double wave_sum_f64(double d) {
  d += row_perm_f64<0xB1>(d);    // quad_perm [1,0,3,2]
  d += row_perm_f64<0x4E>(d);    // quad_perm [2,3,0,1]
  d += row_perm_f64<0x141>(d);   // row_half_mirror
  d += row_perm_f64<0x140>(d);   // row_mirror
  d = lane_pair_sum_f64<16>(d);
  d = lane_pair_sum_f64<32>(d);
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Largest of non-negative floats over the wave, by their bits (which order
// alike, and need no quieting of NaNs first).
__device__ inline float wave_max_f32(float f) {
  uint32_t v = __float_as_uint(f);
#define AQMP_MAXSTEP(C) { const uint32_t o = row_perm_u32<C>(v); v = o > v ? o : v; }
  AQMP_MAXSTEP(0xB1) AQMP_MAXSTEP(0x4E) AQMP_MAXSTEP(0x141) AQMP_MAXSTEP(0x140)
#undef AQMP_MAXSTEP
  uint32_t p, q;
  lane_pair_u32<16>(v, p, q);
  v = p > q ? p : q;
  lane_pair_u32<32>(v, p, q);
  v = p > q ? p : q;
  return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}

// A lane's value, uniform.
__device__ inline double lane_f64(double d, int lane) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Largest of non-negative doubles over the wave, without NaNs, uniform.
template <int X>
__device__ inline double lane_pair_max_f64(double d) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  uint32_t p0, q0, p1, q1;
  lane_pair_u32<X>((uint32_t)u, p0, q0);
  lane_pair_u32<X>((uint32_t)(u >> 32), p1, q1);
  return fmax(__longlong_as_double((long long)(((unsigned long long)p1 << 32) | p0)),
              __longlong_as_double((long long)(((unsigned long long)q1 << 32) | q0)));
}
__device__ inline double wave_max_f64(double d) {
  d = fmax(d, row_perm_f64<0xB1>(d));
  d = fmax(d, row_perm_f64<0x4E>(d));
  d = fmax(d, row_perm_f64<0x141>(d));
  d = fmax(d, row_perm_f64<0x140>(d));
  d = lane_pair_max_f64<16>(d);
  d = lane_pair_max_f64<32>(d);
  const unsigned long long w = (unsigned long long)__double_as_longlong(d);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)w);
  const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(w >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Largest of a row of 16 lanes, in each of them.
__device__ inline unsigned long long row_max_u64(unsigned long long v) {
#define AQMP_RMAX(C) { const unsigned long long o = dpp_u64<C, 0xF>(v); v = o > v ? o : v; }
  AQMP_RMAX(0xB1) AQMP_RMAX(0x4E) AQMP_RMAX(0x141) AQMP_RMAX(0x140)
#undef AQMP_RMAX
  return v;
}

// Smallest of a row of 16 lanes, in each of them, and of the wave, uniform.
__device__ inline int row_min_i32(int v) {
#define AQMP_RMIN(C) { const int o = (int)row_perm_u32<C>((uint32_t)v); v = o < v ? o : v; }
  AQMP_RMIN(0xB1) AQMP_RMIN(0x4E) AQMP_RMIN(0x141) AQMP_RMIN(0x140)
#undef AQMP_RMIN
  return v;
}
__device__ inline int wave_min_i32(int v) {
  v = row_min_i32(v);
  uint32_t p, q;
  lane_pair_u32<16>((uint32_t)v, p, q);
  v = (int)p < (int)q ? (int)p : (int)q;
  lane_pair_u32<32>((uint32_t)v, p, q);
  v = (int)p < (int)q ? (int)p : (int)q;
  return __builtin_amdgcn_readfirstlane(v);
}

typedef double d4 __attribute__((ext_vector_type(4)));
// v_mfma_f64_16x16x4_f64: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; it holds D[l / 16 + 4 r][l % 16], r = 0..3.
__device__ inline d4 mfma64(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// The largest |c| of a lane so far and its atom, the lower of two that differ by
// no more than w (the rounding of the sums).
struct LaneBest {
  double mag = -1.0;
  int atom = 0x7fffffff;
  __device__ inline void take(double c, int a, double w) {
    const double m = fabs(c);
    const bool far = m > mag + w, near = m >= mag - w;
    atom = far ? a : (near && a < atom ? a : atom);
    mag = m > mag ? m : mag;
  }
  // over the wave: the lowest atom of the lanes within w of the largest
  __device__ inline void over_wave(double w) {
    const double m = wave_max_f64(mag);
    atom = wave_min_i32(mag >= m - w ? atom : 0x7fffffff);
    mag = m;
  }
};

}  // namespace aqmp
