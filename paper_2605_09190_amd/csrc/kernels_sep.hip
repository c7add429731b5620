// kernels_sep.hip - whole-level Matching Pursuit of the dense solver at
// N = 32 and 64: one launch runs every node of a level through its whole
// pursuit (Section 2.2 steps (a)-(d), eq. (2)), the residual in registers and
// LDS from the gather to the last step.
//
// The correlation of the residual R (N x N pixels) with all atoms is the
// same c_a = <r, phi_a> as in the step-by-step form, factored through the
// atoms' outer-product shape (Section 2.1): atom (f, p, q) is T_f[p] (x)
// T_f[q], so C_f = T_f R T_f^T holds c_a for every atom of family f, 8 N^3
// operations per node and step for both families instead of the 4 N^4 of the
// unfactored product.  It is made anew from the residual at every step, on
// the matrix cores:
//   BF16 form: every operand split into an FP16 value and an FP16 remainder,
//     hi hi + hi lo + lo hi with FP32 accumulation (the Haar operands are
//     exact signs, see SepOps).  Largest error over ||r|| against FP64 on
//     smooth, edge, noise and pursued blocks: 1.2e-7, where BF16 atoms and
//     residuals give 5.6e-4;
//   FP32 form: FP32 operands and accumulation (1.5e-7; the unfactored FP32
//     product 5.5e-7).
// First product D1[y][q] = sum_x R[y][x] T[q][x], second D2[p][q] =
// sum_y T[p][y] D1[y][q].  A wave owns whole columns q of both: the lane that
// holds D1[16 ty + 4 g + r][q] (the matrix-core output layout, g = lane / 16)
// needs exactly those values as B operand of the second product once its
// k index is taken in the order (ty, g, r), so D1 never leaves the
// registers; the table operands are laid out in that order once per kernel.
//
// Selection: the candidates are all atoms whose |c| is within 2 delta of the
// largest, delta = 2^-13 ||r||.  Either form is within 2^-14.9 ||r|| of the
// FP64 value in the worst case (per product the remainders' rounding and the
// dropped lo lo term, 3 2^-22, and at most 192 FP32 additions, 192 2^-24, of
// sum |T||R|, which Cauchy-Schwarz bounds by the norm): no other atom can be
// the arg-max of the FP64 re-score or tie it.  One atom is left in 98% of the
// steps of an ordinary image.
// The FP64 re-score, the rank-1 update and the norm use the same lane
// patches and the same order of operations as k_select, and the initial
// norm those of k_gather, so the trees, atoms, coefficients and norms are
// those of the step-by-step form bit for bit.
//
// What bounds it: the chain of one node's step (two products, arg-max,
// re-score, update), and the last long nodes of a level.  On three 2048 x
// 2048 planes (36 432 node-steps at N = 64, 74 821 at N = 32) the levels take
// 420 and 193 us; a correlation and a select launch per step took 2 510 and
// 980 us, 32 (N = 64) or 16 times the operations and the residual through
// memory at every step.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

typedef _Float16 sp_h8 __attribute__((ext_vector_type(8)));
typedef float sp_f32x4 __attribute__((ext_vector_type(4)));

// Geometry.  N = 64: the four waves of a workgroup share one node (16
// columns q each), N = 32: a node per wave.  FAMS: family mask (AQMP_DCT |
// AQMP_HAAR, DCT first), BF: BF16 form.
template <int N_, int FAMS_, bool BF_>
struct SepGeo {
  static constexpr int N = N_, K = N * N, FAMS = FAMS_;
  static constexpr bool BF = BF_;
  static constexpr int NFAM = FAMS == 3 ? 2 : 1;
  static constexpr int M = NFAM * K;
  static constexpr int WPN = N == 64 ? 4 : 1;          // waves per node
  static constexpr int NPG = 4 / WPN;                  // nodes per workgroup
  static constexpr int TT = N / 16;                    // 16-wide tiles of a side
  static constexpr int TQ = TT / WPN;                  // q tiles per wave
  static constexpr int VPL = NFAM * TQ * TT * 4;       // correlations per lane
  static constexpr int PW = N / 8, PH = N / 8;         // patch of a lane over the node's waves
  static constexpr int RPW = PH / WPN;                 // patch rows held by one wave
  static constexpr int KS = N / 32;                    // BF16 k-steps (32) of a product
  // LDS rows of the residual, padded by 16 bytes: 16 consecutive rows read
  // at one column offset (16 bytes per lane) fall on all banks once.
  static constexpr int ROWB = (BF ? 2 : 4) * N + 16;
  static constexpr int HALFB = N * ROWB;               // BF16: hi rows, then lo rows
  static constexpr int RBYTES = BF ? 2 * HALFB : HALFB;
  static_assert(RBYTES >= 4 * K, "the gather stages FP32 pixels in the residual buffer");
  // Power of two on the DCT operands of the BF16 form (and on the Haar
  // magnitudes): their FP16 remainders are then normal numbers.
  static constexpr float TS = BF ? 128.f : 1.f;
  static_assert(VPL <= 32, "one mask word per lane");
};

// Whether family f of a dictionary is the Haar one.
template <class G>
__device__ constexpr bool sep_haar(int f) { return G::FAMS == AQMP_HAAR || (G::FAMS == 3 && f == 1); }

// Table operands of a wave, in registers for the whole kernel.  A Haar row is
// one magnitude times -1, 0 or 1: its operands are those signs, exact in BF16
// (no remainder, two products instead of three), and the magnitudes of the
// row and the column multiply the finished correlation.
template <class G, bool BF = G::BF>
struct SepOps;
template <class G>
struct SepOps<G, true> {
  sp_h8 ah[G::NFAM][G::TQ][G::KS], bh[G::NFAM][G::TT][G::KS];   // T[q][x] (first product, B), T[p][y] (second, A)
  sp_h8 al[1][G::TQ][G::KS], bl[1][G::TT][G::KS];               // DCT remainders
  float sp0[G::TQ][4], sp[G::TQ][G::TT];                             // Haar magnitudes: p < 16 by row, then by p tile
};
template <class G>
struct SepOps<G, false> {
  sp_f32x4 a[1][G::TQ][G::TT], b[1][G::TT][G::TT];                  // DCT
  uint2 ha[1][G::TQ][G::TT], hb[1][G::TT][G::TT];                   // Haar signs, BF16 pairs
  float sp0[G::TQ][4], sp[G::TQ][G::TT];
};

__device__ inline sp_h8 sp_hi(const float (&v)[8]) {
  sp_h8 h;
#pragma unroll
  for (int j = 0; j < 8; ++j) h[j] = (_Float16)v[j];
  return h;
}
__device__ inline sp_h8 sp_lo(const float (&v)[8], const sp_h8& h) {
  sp_h8 l;
#pragma unroll
  for (int j = 0; j < 8; ++j) l[j] = (_Float16)(v[j] - (float)h[j]);
  return l;
}

// Two FP32 values -> packed FP16 halves and their packed remainders.  The
// mixed-precision FMA takes FP16 sources and rounds its result to FP16 in
// place, so a value costs one and a half instructions here (BF16 needs
// three: no such FMA exists for it).  op_sel_hi marks an FP16 source, op_sel
// its upper half.
__device__ inline void sp_split2(float a, float b, uint32_t& h, uint32_t& l) {
  const auto p = __builtin_amdgcn_cvt_pkrtz(a, b);
  __builtin_memcpy(&h, &p, 4);
  __asm__("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(l) : "v"(h), "v"(a));
  __asm__("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(l) : "v"(h), "v"(b));
}
// The same for a * s and b * s (s a power of two).
__device__ inline void sp_split2_scaled(float a, float b, float s, uint32_t& h, uint32_t& l) {
  __asm__("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(a), "v"(s));
  __asm__("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(b), "v"(s));
  __asm__("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(l) : "v"(a), "v"(s), "v"(h));
  __asm__("v_fma_mixhi_f16 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(l) : "v"(b), "v"(s), "v"(h));
}

__device__ inline float sp_sign(double v) { return v > 0.0 ? 1.f : (v < 0.0 ? -1.f : 0.f); }
__device__ inline uint2 sp_pack4(const float (&v)[4]) {   // exact in BF16
  return make_uint2((__float_as_uint(v[0]) >> 16) | (__float_as_uint(v[1]) & 0xFFFF0000u),
                    (__float_as_uint(v[2]) >> 16) | (__float_as_uint(v[3]) & 0xFFFF0000u));
}
__device__ inline float sp_unpack(const uint2& u, int r) {
  const uint32_t w = r < 2 ? u.x : u.y;
  return __uint_as_float((r & 1) ? (w & 0xFFFF0000u) : (w << 16));
}

template <class G>
__device__ inline void sep_load_ops(SepOps<G>& T, const double* __restrict__ tab, int wq) {
  constexpr int N = G::N;
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
#pragma unroll
  for (int f = 0; f < G::NFAM; ++f) {
    const double* tf = tab + (size_t)f * G::K;
    auto entry = [&](int row, int col) -> float {
      const double v = tf[row * N + col];
      return sep_haar<G>(f) ? sp_sign(v) : (float)v * G::TS;
    };
    if constexpr (G::BF) {
#pragma unroll
      for (int i = 0; i < G::TQ; ++i)
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          float v[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] = entry(16 * (wq * G::TQ + i) + m, 32 * ks + 8 * g + j);
          T.ah[f][i][ks] = sp_hi(v);
          if (!sep_haar<G>(f)) T.al[0][i][ks] = sp_lo(v, T.ah[f][i][ks]);
        }
#pragma unroll
      for (int tp = 0; tp < G::TT; ++tp)
#pragma unroll
        for (int ks = 0; ks < G::KS; ++ks) {
          float v[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) v[j] = entry(16 * tp + m, 32 * ks + 16 * (j >> 2) + 4 * g + (j & 3));
          T.bh[f][tp][ks] = sp_hi(v);
          if (!sep_haar<G>(f)) T.bl[0][tp][ks] = sp_lo(v, T.bh[f][tp][ks]);
        }
    } else {
#pragma unroll
      for (int i = 0; i < G::TQ; ++i)
#pragma unroll
        for (int c = 0; c < G::TT; ++c) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = entry(16 * (wq * G::TQ + i) + m, 16 * c + 4 * g + r);
          if (sep_haar<G>(f)) T.ha[0][i][c] = sp_pack4(v);
          else T.a[0][i][c] = sp_f32x4{v[0], v[1], v[2], v[3]};
        }
#pragma unroll
      for (int tp = 0; tp < G::TT; ++tp)
#pragma unroll
        for (int ty = 0; ty < G::TT; ++ty) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = entry(16 * tp + m, 16 * ty + 4 * g + r);
          if (sep_haar<G>(f)) T.hb[0][tp][ty] = sp_pack4(v);
          else T.b[0][tp][ty] = sp_f32x4{v[0], v[1], v[2], v[3]};
        }
    }
    if (sep_haar<G>(f)) {
      // a row's magnitude is its value at the first pixel of its support
      auto mag = [&](int row) -> float {
        int at = 0;
        if (row > 0) {
          const int top = 1 << (31 - __builtin_clz((unsigned)row));
          at = (row - top) * (N / top);
        }
        return (float)tf[row * N + at];
      };
#pragma unroll
      for (int i = 0; i < G::TQ; ++i) {
        const float mq = mag(16 * (wq * G::TQ + i) + m);
#pragma unroll
        for (int r = 0; r < 4; ++r) T.sp0[i][r] = mag(4 * g + r) * mq * (G::TS * G::TS);
#pragma unroll
        for (int tp = 1; tp < G::TT; ++tp) T.sp[i][tp] = mag(16 * tp) * mq * (G::TS * G::TS);   // one scale from row 16 up to the next power of two
      }
    }
  }
}

// All correlations of the residual in sR with the wave's columns q:
// C[f][i][tp][r] = c of atom (f, p = 16 tp + 4 g + r, q = 16 (TQ wq + i) + m).
template <class G>
__device__ inline void sep_correlate(const char* sR, const SepOps<G>& T, sp_f32x4 (&C)[G::NFAM][G::TQ][G::TT]) {
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  sp_f32x4 D[G::NFAM][G::TQ][G::TT];
#pragma unroll
  for (int f = 0; f < G::NFAM; ++f)
#pragma unroll
    for (int i = 0; i < G::TQ; ++i)
#pragma unroll
      for (int t = 0; t < G::TT; ++t) D[f][i][t] = C[f][i][t] = sp_f32x4{0.f, 0.f, 0.f, 0.f};
  const char* base = sR + m * G::ROWB + 16 * g;
  if constexpr (G::BF) {
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks)
#pragma unroll
      for (int ty = 0; ty < G::TT; ++ty) {
        const sp_h8 rh = *(const sp_h8*)(base + 16 * ty * G::ROWB + 64 * ks);
        const sp_h8 rl = *(const sp_h8*)(base + G::HALFB + 16 * ty * G::ROWB + 64 * ks);
#pragma unroll
        for (int pr = 0; pr < 3; ++pr)
#pragma unroll
          for (int f = 0; f < G::NFAM; ++f)
#pragma unroll
            for (int i = 0; i < G::TQ; ++i) {
              if (pr == 1 && sep_haar<G>(f)) continue;   // no remainder
              D[f][i][ty] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pr == 2 ? rl : rh, pr == 1 ? T.al[0][i][ks] : T.ah[f][i][ks],
                                                                    D[f][i][ty], 0, 0, 0);
            }
      }
#pragma unroll
    for (int f = 0; f < G::NFAM; ++f)
#pragma unroll
      for (int ks = 0; ks < G::KS; ++ks) {
        sp_h8 zh[G::TQ], zl[G::TQ];
#pragma unroll
        for (int i = 0; i < G::TQ; ++i) {
          uint32_t h[4], l[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const sp_f32x4& d = D[f][i][2 * ks + (j >> 1)];
            sp_split2(d[2 * (j & 1)], d[2 * (j & 1) + 1], h[j], l[j]);
          }
          __builtin_memcpy(&zh[i], h, 16);
          __builtin_memcpy(&zl[i], l, 16);
        }
#pragma unroll
        for (int pr = 0; pr < 3; ++pr)
#pragma unroll
          for (int tp = 0; tp < G::TT; ++tp)
#pragma unroll
            for (int i = 0; i < G::TQ; ++i) {
              if (pr == 1 && sep_haar<G>(f)) continue;
              C[f][i][tp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pr == 1 ? T.bl[0][tp][ks] : T.bh[f][tp][ks],
                                                                    pr == 2 ? zl[i] : zh[i], C[f][i][tp], 0, 0, 0);
            }
      }
  } else {
#pragma unroll
    for (int c = 0; c < G::TT; ++c)
#pragma unroll
      for (int ty = 0; ty < G::TT; ++ty) {
        const sp_f32x4 rv = *(const sp_f32x4*)(base + 16 * ty * G::ROWB + 64 * c);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int f = 0; f < G::NFAM; ++f)
#pragma unroll
            for (int i = 0; i < G::TQ; ++i) {
              const float tv = sep_haar<G>(f) ? sp_unpack(T.ha[0][i][c], r) : T.a[0][i][c][r];
              D[f][i][ty] = __builtin_amdgcn_mfma_f32_16x16x4f32(rv[r], tv, D[f][i][ty], 0, 0, 0);
            }
      }
#pragma unroll
    for (int f = 0; f < G::NFAM; ++f)
#pragma unroll
      for (int ty = 0; ty < G::TT; ++ty)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int tp = 0; tp < G::TT; ++tp)
#pragma unroll
            for (int i = 0; i < G::TQ; ++i) {
              const float tv = sep_haar<G>(f) ? sp_unpack(T.hb[0][tp][ty], r) : T.b[0][tp][ty][r];
              C[f][i][tp] = __builtin_amdgcn_mfma_f32_16x16x4f32(tv, D[f][i][ty][r], C[f][i][tp], 0, 0, 0);
            }
  }
#pragma unroll
  for (int f = 0; f < G::NFAM; ++f)
    if (sep_haar<G>(f)) {
#pragma unroll
      for (int i = 0; i < G::TQ; ++i)
#pragma unroll
        for (int tp = 0; tp < G::TT; ++tp)
#pragma unroll
          for (int r = 0; r < 4; ++r) C[f][i][tp][r] *= tp == 0 ? T.sp0[i][r] : T.sp[i][tp];
    }
}

// Orders a node's LDS writes before its other lanes' reads: a workgroup
// barrier that waits for LDS only (no global access is shared between the
// waves), or, for a node held by one wave, the wave's own order.
template <int WPN>
__device__ inline void sep_sync() {
  if constexpr (WPN > 1) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  } else {
    wave_sync();
  }
}

// FP64 1D tables in LDS: the DCT as it is; a Haar row is one magnitude
// times -1, 0 or 1 (exact products), kept as FP32 signs and one FP64
// magnitude per scale (row 0, then rows [2^j, 2^(j+1))).
template <class G>
struct SepTab {
  double dct[(G::FAMS & AQMP_DCT) ? G::K : 1];
  float sgn[(G::FAMS & AQMP_HAAR) ? G::K : 1];
  double mag[8];
};

__device__ inline int sep_haar_scale(int p) { return p == 0 ? 0 : 32 - __builtin_clz((unsigned)p); }

template <class G>
__device__ inline void sep_load_tab(SepTab<G>& S, const double* __restrict__ tab) {
  const int tid = threadIdx.x;
  if constexpr ((G::FAMS & AQMP_DCT) != 0)
    for (int i = tid; i < G::K; i += 256) S.dct[i] = tab[i];
  if constexpr ((G::FAMS & AQMP_HAAR) != 0) {
    const double* h = tab + (G::FAMS == 3 ? G::K : 0);
    for (int i = tid; i < G::K; i += 256) S.sgn[i] = h[i] > 0.0 ? 1.f : (h[i] < 0.0 ? -1.f : 0.f);
    // the first row of a scale starts at pixel 0
    if (tid < 8) {
      const int row = tid == 0 ? 0 : 1 << (tid - 1);
      S.mag[tid] = row < G::N ? h[row * G::N] : 0.0;
    }
  }
}

// CNT consecutive FP64 entries of row p of family f (uniform f, p).
template <class G, int CNT>
__device__ inline void sep_row(const SepTab<G>& S, int f, int p, int at, double (&v)[CNT]) {
  const bool haar = G::FAMS == AQMP_HAAR || (G::FAMS == 3 && f == 1);
  if (haar) {
    if constexpr ((G::FAMS & AQMP_HAAR) != 0) {
      const double mg = S.mag[sep_haar_scale(p)];
#pragma unroll
      for (int j = 0; j < CNT; ++j) v[j] = (double)S.sgn[p * G::N + at + j] * mg;
    }
  } else {
    if constexpr ((G::FAMS & AQMP_DCT) != 0) {
#pragma unroll
      for (int j = 0; j < CNT; ++j) v[j] = S.dct[p * G::N + at + j];
    }
  }
}

__device__ inline double sep_bcast_f64(double d) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The table operands of every thread of a workgroup, 16 bytes at a time in
// thread order, made once with the dictionary (making them in the pursuit
// took about 2 000 instructions per launch).
template <class G>
struct SepOpsBuf {
  static constexpr int E = (int)((sizeof(SepOps<G>) + 15) / 16);
  union U {
    SepOps<G> ops;
    uint4 w[E];
    __device__ U() {}
  };
};

template <int N, int FAMS, bool BF>
__global__ __launch_bounds__(256) void k_sep_ops(const double* __restrict__ tab, uint4* __restrict__ out) {
  using B = SepOpsBuf<SepGeo<N, FAMS, BF>>;
  typename B::U u;
#pragma unroll
  for (int e = 0; e < B::E; ++e) u.w[e] = make_uint4(0u, 0u, 0u, 0u);
  sep_load_ops<SepGeo<N, FAMS, BF>>(u.ops, tab, N == 64 ? (int)(threadIdx.x >> 6) : 0);
#pragma unroll
  for (int e = 0; e < B::E; ++e) out[e * 256 + threadIdx.x] = u.w[e];
}

template <int N, int FAMS, bool BF>
__global__ __launch_bounds__(256, 2) void k_pursuit_sep(const JobDev* __restrict__ jobs, LevelDev lv,
                                                        const int32_t* __restrict__ count_ptr,
                                                        int32_t* __restrict__ queue, int32_t lg,
                                                        const double* __restrict__ tab,
                                                        const uint4* __restrict__ ops) {
  using G = SepGeo<N, FAMS, BF>;
  constexpr int K = G::K, WPN = G::WPN, NPG = G::NPG, PW = G::PW, PH = G::PH, RPW = G::RPW, VPL = G::VPL;
  __shared__ __attribute__((aligned(16))) char sRes[NPG][G::RBYTES];
  __shared__ __attribute__((aligned(16))) SepTab<G> sTab;
  __shared__ __attribute__((aligned(16))) uint4 sTop[WPN > 1 ? 4 : 1];            // per wave: largest |c|, its atom, several candidates
  __shared__ __attribute__((aligned(16))) double sPart[WPN > 1 ? 2 : 1][WPN > 1 ? PH : 1][WPN > 1 ? 64 : 1];
  __shared__ uint32_t sMask[WPN > 1 ? 256 : 1];
  __shared__ double sRed[4];
  __shared__ int sNode[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = WPN > 1 ? wv : 0;                       // wave within the node
  const int grp = WPN > 1 ? 0 : wv;                      // node slot of the workgroup
  char* sR = sRes[grp];
  typename SepOpsBuf<G>::U opu;
#pragma unroll
  for (int i = 0; i < SepOpsBuf<G>::E; ++i) opu.w[i] = ops[i * 256 + tid];
  const SepOps<G>& T = opu.ops;
  sep_load_tab<G>(sTab, tab);
  __syncthreads();
  const int count = *count_ptr;
  const double inv_n = 1.0 / N;
  const int py = (lane >> 3) * PH + wq * RPW;            // first pixel of the lane's rows
  const int px = (lane & 7) * PW;
  // The first nodes are dealt out in order, the others by the queues: queue
  // k holds every kQueues-th node after the first ones.
  const int q0 = (int)gridDim.x * NPG, qk = (int)blockIdx.x % kQueues;
  int par = 0;                                           // sPart buffer in use
  int node = (int)blockIdx.x * NPG + grp;
  while (node < count) {
    const int jidx = lv.job[node];
    const int bx = lv.x0[node], by = lv.y0[node];
    const JobDev jl = jobs[jidx];
    const double eps2 = sep_bcast_f64(jobs[jidx].eps2[lg]);
    const int kmax = __builtin_amdgcn_readfirstlane(jobs[jidx].k[lg]);
    // ---- gather: FP64 norm in the lane layout and order of k_gather, FP32
    // pixels through LDS to the patches ----
    double e;
    {
      float* st = (float*)sR;
      if constexpr (WPN > 1) {
        constexpr int GP = 4;                            // 4 x 4 pixels per thread
        const int gy = (tid / (N / GP)) * GP, gx = (tid % (N / GP)) * GP;
        double pv[GP][GP];
#pragma unroll
        for (int dy = 0; dy < GP; ++dy) job_pixels<GP>(jl, by + gy + dy, bx + gx, pv[dy]);
        double ep = 0.0;
#pragma unroll
        for (int dy = 0; dy < GP; ++dy)
#pragma unroll
          for (int dx = 0; dx < GP; ++dx) {
            const double v = pv[dy][dx];
            st[(gy + dy) * N + gx + dx] = (float)v;
            ep += v * v;
          }
        e = group_sum<256>(ep, sRed);
      } else {
        constexpr int GP = 2;                            // 2 x 2 pixels per thread of four virtual waves
        double ev[4];
        double pv[4][GP][GP];
#pragma unroll
        for (int vw = 0; vw < 4; ++vw) {
          const int lt = 64 * vw + lane, gy = (lt / (N / GP)) * GP, gx = (lt % (N / GP)) * GP;
#pragma unroll
          for (int dy = 0; dy < GP; ++dy) job_pixels<GP>(jl, by + gy + dy, bx + gx, pv[vw][dy]);
        }
#pragma unroll
        for (int vw = 0; vw < 4; ++vw) {
          const int lt = 64 * vw + lane, gy = (lt / (N / GP)) * GP, gx = (lt % (N / GP)) * GP;
          ev[vw] = 0.0;
#pragma unroll
          for (int dy = 0; dy < GP; ++dy)
#pragma unroll
            for (int dx = 0; dx < GP; ++dx) {
              const double v = pv[vw][dy][dx];
              st[(gy + dy) * N + gx + dx] = (float)v;
              ev[vw] += v * v;
            }
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) ev[vw] += __shfl_xor(ev[vw], off, 64);
        }
        e = (ev[0] + ev[1]) + (ev[2] + ev[3]);
      }
    }
    e = sep_bcast_f64(e);
    sep_sync<WPN>();
    float r[RPW][PW];
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int j = 0; j < PW; ++j) r[i][j] = ((const float*)sR)[(py + i) * N + px + j];
    sep_sync<WPN>();
    // the node after this one: taken here, needed at the end
    int ahead = 0;
    if (WPN > 1 ? tid == 0 : lane == 0) ahead = atomicAdd(queue + qk * kQueuePad, 1);
    // Scale of the operand rows, a power of two.  FP16 halves: ||r|| goes to
    // [2^7, 2^8), so that the first product (at most 2^15) and the
    // remainders stay inside FP16's range.  FP32: 1 unless the plane's
    // values are far from the usual range.
    auto scale_of = [](double en) -> float {
      const int ex = (int)((unsigned long long)__double_as_longlong(en) >> 52) - 1023;
      int sh = ex >> 1;
      if constexpr (BF) sh -= 7;
      else if (ex >= -40 && ex < 80) return 1.f;
      sh = sh < -120 ? -120 : (sh > 120 ? 120 : sh);
      return __uint_as_float((uint32_t)(127 - sh) << 23);
    };
    float sc = scale_of(e);
    auto put_rows = [&]() {                              // the lane's pixels into the operand rows
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        char* row = sR + (py + i) * G::ROWB;
        if constexpr (BF) {
          uint32_t h[PW / 2], l[PW / 2];
#pragma unroll
          for (int j = 0; j < PW / 2; ++j) sp_split2_scaled(r[i][2 * j], r[i][2 * j + 1], sc, h[j], l[j]);
          if constexpr (PW == 8) {
            *(uint4*)(row + 2 * px) = make_uint4(h[0], h[1], h[2], h[3]);
            *(uint4*)(row + G::HALFB + 2 * px) = make_uint4(l[0], l[1], l[2], l[3]);
          } else {
            *(uint2*)(row + 2 * px) = make_uint2(h[0], h[1]);
            *(uint2*)(row + G::HALFB + 2 * px) = make_uint2(l[0], l[1]);
          }
        } else {
#pragma unroll
          for (int j = 0; j < PW; j += 4) {
            sp_f32x4 v{r[i][j], r[i][j + 1], r[i][j + 2], r[i][j + 3]};
            if (sc != 1.f) v *= sc;
            *(sp_f32x4*)(row + 4 * (px + j)) = v;
          }
        }
      }
    };
    uint8_t st = ST_RUN;
    if (e < eps2)
      st = ST_ACC;
    else if (kmax <= 0)
      st = ST_SPARSE;
    int t = 0;
    int rec_i = 0;
    double rec_c = 0.0;
    const size_t rec0 = (size_t)node * lv.kmax;
    if (st == ST_RUN) put_rows();
    sep_sync<WPN>();
    while (st == ST_RUN) {
      if (!(e > 0.0 && e < __builtin_inf())) {           // a zero residual, or undefined pixels: nothing to select
        st = ST_ZERO;
        break;
      }
      // ---- correlations; the wave's atoms within 2 delta of its largest ----
      uint32_t mask = 0u;                                // bit VPL - 1 - j: value j is within
      float mx;
      const float win = __builtin_amdgcn_sqrtf((float)(e * ((double)sc * (double)sc))) * (1.0001f * 0x1p-12f * G::TS * G::TS);
      {
        sp_f32x4 C[G::NFAM][G::TQ][G::TT];
        sep_correlate<G>(sR, T, C);
        if constexpr (G::NFAM == 2) {
          // the second family's constant atom equals the first's, which wins the tie
          if (wq == 0 && lane == 0) C[1][0][0][0] = 0.f;
        }
        auto val = [&](int j) -> float {
          return C[j / (4 * G::TT * G::TQ)][(j / (4 * G::TT)) % G::TQ][(j >> 2) % G::TT][j & 3];
        };
        float m0 = 0.f, m1 = 0.f;
#pragma unroll
        for (int j = 0; j < VPL; j += 4) {
          m0 = fmaxf(fmaxf(fabsf(val(j)), fabsf(val(j + 1))), m0);
          m1 = fmaxf(fmaxf(fabsf(val(j + 2)), fabsf(val(j + 3))), m1);
        }
        mx = wave_max_f32(fmaxf(m0, m1));
        // the sign of thr - |c| into the mask: two instructions per value
        const float thr = mx - win;
#pragma unroll
        for (int j = 0; j < VPL; ++j)
          mask = __builtin_amdgcn_alignbit(mask, __float_as_uint(thr - fabsf(val(j))), 31);
        if (!(mx > 0.f && mx < __builtin_inff())) mask = 0u;   // undefined sums: nothing to compare
      }
      auto atom_of = [&](int w, int l, int bit) -> int {   // wave of the node, lane, bit of its mask
        const int j = VPL - 1 - bit, f = j / (4 * G::TT * G::TQ), i = (j / (4 * G::TT)) % G::TQ, tp = (j >> 2) % G::TT;
        return f * K + (16 * (w * G::TQ + i) + (l & 15)) * N + 16 * tp + 4 * (l >> 4) + (j & 3);
      };
      const unsigned long long near = __ballot(mask != 0u);
      bool several = __popcll(near) != 1 || __ballot((mask & (mask - 1u)) != 0u) != 0ull;
      int cand = 0;
      {
        const int l = near ? __builtin_ctzll(near) : 0;
        const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)mask, l);
        cand = atom_of(wq, l, bits ? __builtin_ctz(bits) : 0);
      }
      uint32_t wsel = 1u;                                // waves with a candidate
      if constexpr (WPN > 1) {
        if (lane == 0) sTop[wv] = make_uint4(__float_as_uint(mx), (uint32_t)cand, several ? 1u : 0u, 0u);
        sep_sync<WPN>();
        float wm[4];
        uint32_t sev = 0u;
#pragma unroll
        for (int w = 0; w < 4; ++w) wm[w] = __uint_as_float(sTop[w].x);
        mx = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
        const float thr = mx - win;
        wsel = 0u;
#pragma unroll
        for (int w = 0; w < 4; ++w) wsel |= wm[w] >= thr ? 1u << w : 0u;
        wsel = (uint32_t)__builtin_amdgcn_readfirstlane((int)wsel);
        const uint4 only = sTop[wsel ? __builtin_ctz(wsel) : 0];
        cand = __builtin_amdgcn_readfirstlane((int)only.y);
        sev = (uint32_t)__builtin_amdgcn_readfirstlane((int)only.z);
        several = sev != 0u || (wsel & (wsel - 1u)) != 0u;
        mx = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(mx)));
      }
      // ---- FP64 re-score (k_select's patches and order of operations) ----
      double tq[PW], tp8[PH];
      auto rescore = [&](int at) -> double {
        const int f = at / K, q = (at % K) / N, p = at % N;
        const bool dc = p == 0 && q == 0;
        sep_row<G, PW>(sTab, f, q, px, tq);
        sep_row<G, PH>(sTab, f, p, (lane >> 3) * PH, tp8);
        double sr[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
          sr[i] = 0.0;
          if (dc) {
#pragma unroll
            for (int j = 0; j < PW; ++j) sr[i] += (double)r[i][j];
          } else {
#pragma unroll
            for (int j = 0; j < PW; ++j) sr[i] = fma((double)r[i][j], tq[j], sr[i]);
          }
        }
        double all[PH];
        if constexpr (WPN > 1) {
          // the row sums of the node's four waves
#pragma unroll
          for (int i = 0; i < RPW; ++i) sPart[par][wq * RPW + i][lane] = sr[i];
          sep_sync<WPN>();
#pragma unroll
          for (int i = 0; i < PH; ++i) all[i] = sPart[par][i][lane];
          par ^= 1;
        } else {
#pragma unroll
          for (int i = 0; i < PH; ++i) all[i] = sr[i];
        }
        double part = 0.0;
        if (dc) {
#pragma unroll
          for (int i = 0; i < PH; ++i) part += all[i];
          part *= inv_n;
        } else {
#pragma unroll
          for (int i = 0; i < PH; ++i) part = fma(tp8[i], all[i], part);
        }
        return wave_sum_f64(part);
      };
      int atom = -1;
      double coef = 0.0, mag = -1.0;
      if (!several && mx < __builtin_inff()) {
        coef = rescore(cand);
        mag = fabs(coef);
        atom = cand;
      } else if (mx < __builtin_inff()) {
        // several atoms within the window: every one of them, lowest index on
        // ties (a wave's mask is relative to its own largest: no fewer atoms)
        if constexpr (WPN > 1) {
          sMask[tid] = mask;
          sep_sync<WPN>();
        }
        for (int w = 0; w < WPN; ++w) {
          if (!((wsel >> w) & 1u)) continue;
          const uint32_t mw = WPN > 1 ? sMask[64 * w + lane] : mask;
          unsigned long long lanes = __ballot(mw != 0u);
          while (lanes) {
            const int l = __builtin_ctzll(lanes);
            lanes &= lanes - 1ull;
            uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)mw, l);
            while (bits) {
              const int bit = __builtin_ctz(bits);
              bits &= bits - 1u;
              const int at = atom_of(w, l, bit);
              const double c0 = rescore(at), m0 = fabs(c0);
              if (m0 > mag || (m0 == mag && at < atom)) {
                mag = m0;
                coef = c0;
                atom = at;
              }
            }
          }
        }
        if (atom >= 0) {
          const int f = atom / K, q = (atom % K) / N, p = atom % N;
          sep_row<G, PW>(sTab, f, q, px, tq);
          sep_row<G, PH>(sTab, f, p, (lane >> 3) * PH, tp8);
        }
      }
      if (atom < 0 || mag == 0.0) {
        st = ST_ZERO;
        break;
      }
      // ---- rank-1 update, norm, record, stop test ----
      const bool dc = (atom % K) == 0;
      double eh[RPW];
      {
        double ty[RPW];
        if constexpr (WPN > 1) {
#pragma unroll
          for (int i = 0; i < RPW; ++i) {
            double v = tp8[i];
#pragma unroll
            for (int w = 1; w < 4; ++w) v = wq == w ? tp8[w * RPW + i] : v;
            ty[i] = v;
          }
        } else {
#pragma unroll
          for (int i = 0; i < RPW; ++i) ty[i] = tp8[i];
        }
        if (dc) {
#pragma unroll
          for (int i = 0; i < RPW; ++i) ty[i] = inv_n;
#pragma unroll
          for (int j = 0; j < PW; ++j) tq[j] = 1.0;
        }
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
          eh[i] = 0.0;
#pragma unroll
          for (int j = 0; j < PW; ++j) {
            const double phi = ty[i] * tq[j];
            const float rn = (float)fma(-coef, phi, (double)r[i][j]);
            r[i][j] = rn;
            eh[i] = fma((double)rn, (double)rn, eh[i]);
          }
        }
      }
      if constexpr (BF) {
        // scaled by the norm to come, e - c^2 but for the rounding of the residual
        const double ep = fma(-coef, coef, e), lo = e * 0x1p-30;
        sc = scale_of(ep > lo ? ep : lo);
      }
      put_rows();
      double ew = 0.0;
      if constexpr (WPN > 1) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) sPart[par][wq * RPW + i][lane] = eh[i];
        sep_sync<WPN>();
#pragma unroll
        for (int i = 0; i < PH; ++i) ew += sPart[par][i][lane];
        par ^= 1;
      } else {
        sep_sync<WPN>();
#pragma unroll
        for (int i = 0; i < PH; ++i) ew += eh[i];
      }
      e = wave_sum_f64(ew);
      if constexpr (BF) {
        const double es = e * ((double)sc * (double)sc);
        if (!(es >= 0x1p8 && es < 0x1p18) && e > 0.0 && e < __builtin_inf()) {   // the guess was off: once more
          sc = scale_of(e);
          sep_sync<WPN>();
          put_rows();
          sep_sync<WPN>();
        }
      }
      if (lane == (t & 63)) {
        rec_i = atom;
        rec_c = coef;
      }
      ++t;
      if ((t & 63) == 0 && wq == 0) {
        lv.rec_idx[rec0 + t - 64 + lane] = rec_i;
        lv.rec_coef[rec0 + t - 64 + lane] = rec_c;
      }
      if (e < eps2)
        st = ST_ACC;
      else if (t >= kmax)
        st = ST_SPARSE;
    }
    if (wq == 0) {
      if (lane < (t & 63)) {
        lv.rec_idx[rec0 + (t & ~63) + lane] = rec_i;
        lv.rec_coef[rec0 + (t & ~63) + lane] = rec_c;
      }
      if (lane == 0) {
        lv.e[node] = e;
        lv.t[node] = t;
        lv.st[node] = st;
      }
    }
    // The next node, through LDS so that every lane takes the same value.
    if (WPN > 1 ? tid == 0 : lane == 0) sNode[grp] = q0 + ahead * kQueues + qk;
    sep_sync<WPN>();
    node = __builtin_amdgcn_readfirstlane(sNode[grp]);
    sep_sync<WPN>();
  }
}

template <int N, int FAMS, bool BF>
hipError_t launch_sep_n(const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue, int64_t cap,
                        const double* tab, const void* ops, hipStream_t s) {
  using G = SepGeo<N, FAMS, BF>;
  // Nodes come from a counter, so the grid is as many workgroups as are
  // resident at once (at most one per NPG nodes of the level).
  int dev = 0, n_cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pursuit_sep<N, FAMS, BF>, 256, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  int64_t wgs = (cap + G::NPG - 1) / G::NPG;
  if (wgs > (int64_t)n_cus * per_cu) wgs = (int64_t)n_cus * per_cu;
  if (wgs < 1) wgs = 1;
  hipLaunchKernelGGL((k_pursuit_sep<N, FAMS, BF>), dim3((unsigned)wgs), dim3(256), 0, s, jobs, lv, count, queue,
                     ilog2(N), tab, (const uint4*)ops);
  return hipGetLastError();
}

template <int N, int FAMS, bool BF>
hipError_t launch_sep_ops_n(const double* tab, void* out, hipStream_t s) {
  hipLaunchKernelGGL((k_sep_ops<N, FAMS, BF>), dim3(1), dim3(256), 0, s, tab, (uint4*)out);
  return hipGetLastError();
}

}  // namespace

// Calls CALL with NN, FF, BB set for a block size, family mask and precision.
#define AQMP_SEP_F(NN_, CALL)                                                                              \
  {                                                                                                        \
    constexpr int NN = NN_;                                                                                \
    if (precision == AQMP_PREC_BF16) {                                                                     \
      constexpr bool BB = true;                                                                            \
      switch (families) {                                                                                  \
        case 1: { constexpr int FF = 1; CALL; }                                                            \
        case 2: { constexpr int FF = 2; CALL; }                                                            \
        case 3: { constexpr int FF = 3; CALL; }                                                            \
      }                                                                                                    \
    } else {                                                                                               \
      constexpr bool BB = false;                                                                           \
      switch (families) {                                                                                  \
        case 1: { constexpr int FF = 1; CALL; }                                                            \
        case 2: { constexpr int FF = 2; CALL; }                                                            \
        case 3: { constexpr int FF = 3; CALL; }                                                            \
      }                                                                                                    \
    }                                                                                                      \
  }
#define AQMP_SEP(CALL)             \
  switch (n) {                     \
    case 32: AQMP_SEP_F(32, CALL) break; \
    case 64: AQMP_SEP_F(64, CALL) break; \
  }

size_t sep_ops_bytes(int n, int precision, uint32_t families) {
  AQMP_SEP(return sizeof(uint4) * 256 * (size_t)(SepOpsBuf<SepGeo<NN, FF, BB>>::E))
  return 0;
}

hipError_t launch_sep_ops(int n, int precision, uint32_t families, const double* tab, void* out, hipStream_t s) {
  AQMP_SEP(return (launch_sep_ops_n<NN, FF, BB>(tab, out, s)))
  return hipErrorInvalidValue;
}

hipError_t launch_pursuit_sep(int n, int precision, uint32_t families, const JobDev* jobs, LevelDev lv,
                              const int32_t* count, int32_t* queue, int64_t cap, const double* tab, const void* ops,
                              hipStream_t s) {
  AQMP_SEP(return (launch_sep_n<NN, FF, BB>(jobs, lv, count, queue, cap, tab, ops, s)))
  return hipErrorInvalidValue;
}

}  // namespace aqmp
