// kernels_sep.hip - whole-level Matching Pursuit of the dense solver at
// N = 32 and 64: one launch runs every node of a level through its whole
// pursuit (Section 2.2 steps (a)-(d), eq. (2)), the residual in registers and
// LDS from the gather to the last step.
//
// The correlation of the residual R (N x N pixels) with all atoms is the
// same c_a = <r, phi_a> as in the step-by-step form, factored through the
// atoms' outer-product shape (Section 2.1): atom (f, p, q) is T_f[p] (x)
// T_f[q], so C_f = T_f R T_f^T holds c_a for every atom of family f, 8 N^3
// operations for both families instead of the 4 N^4 of the unfactored
// product.  Matrix cores, every operand split into an FP16 value and an FP16
// remainder, hi hi + hi lo + lo hi with FP32 accumulation (the Haar operands
// are exact signs, see sep_make_ops).  First product D1[y][q] = sum_x R[y][x]
// T[q][x], second D2[p][q] = sum_y T[p][y] D1[y][q].  A wave owns whole
// columns q of both: the lane that holds D1[16 ty + 4 g + r][q] (the
// matrix-core output layout, g = lane / 16) needs exactly those values as B
// operand of the second product once its k index is taken in the order (ty,
// g, r), so D1 never leaves the registers; the table operands and the rows of
// R are laid out in that order, and one table serves both products.
//
// A step with atom (f, p, q) and coefficient c takes c phi from the residual,
// so every correlation loses c <phi, phi'>: c for the atom itself, 0 for the
// rest of its family (an orthonormal basis), c X[p][p'] X[q][q'] for the other
// family, X the 1D products <T_0[p], T_1[p']>.  The correlations are therefore
// carried in FP32 registers from step to step (2 operations per atom of one
// family instead of 4 N per atom of both) and made anew from the residual
// when its norm has halved, or after at most 64 steps.  Largest error over
// ||r|| against FP64, whole pursuits over blocks of 35 planes (51 to 1 822
// pixels wide, k to 40), every FP32 sum taken one term after the other: 7.3e-7
// at N = 32, 6.2e-7 at N = 64; the unfactored product of every step has 2.5e-6
// and 2.3e-6 with FP32 operands (and, summed in blocks, 5.6e-4 with BF16 atoms
// and residuals).  Both forms run this one kernel.
//
// Selection: the candidates are all atoms whose |c| is within 2 delta of the
// largest, delta = 2^-14 ||r'||, r' the residual of the last product.  A
// fresh correlation is within 2^-14.9 ||r'|| of the FP64 value in the worst
// case (the remainders' rounding and the dropped lo lo term, 3 2^-22 in the
// first product and 5 2^-22 in the second, whose operand is split by
// truncation, and at most 192 FP32 additions in either, 192 2^-24, of sum
// |T||R|, which Cauchy-Schwarz bounds by the norm), and a step adds at most 6 2^-24 ||r'||
// (roundings of c, X, two products, the sum, and of the stored residual), 64
// of them 2^-15.4 ||r'||: no other atom can be the arg-max of the FP64
// re-score or tie it.  One atom is left in 98% of the steps of an ordinary
// image.  (Many: see kSepMany.)
// The FP64 re-score, the rank-1 update and the norm use the same lane
// patches and the same order of operations as k_select, and the initial
// norm those of k_gather, so the trees, atoms, coefficients and norms are
// those of the step-by-step form bit for bit.
//
// What bounds it: the chain of one node's step (re-score 1 460 cycles, update
// of residual and correlations 1 060, arg-max 720, norm and stop test 700;
// correlations anew 4 700, 1.9 times a node), and the last long nodes of a
// level.  On three 2048 x 2048 planes (36 432 node-steps at N = 64, 74 821 at
// N = 32) the levels take 233 and 87 us; with the correlations made anew at
// every step 444 and 191 us, and with a correlation and a select launch per
// step 2 510 and 980 us.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

typedef _Float16 sp_h8 __attribute__((ext_vector_type(8)));
typedef float sp_f32x4 __attribute__((ext_vector_type(4)));
typedef float sp_f32x16 __attribute__((ext_vector_type(16)));

// Geometry.  N = 64: the four waves of a workgroup share one node (16
// columns q each), N = 32: a node per wave.  FAMS: family mask (AQMP_DCT |
// AQMP_HAAR, DCT first).
template <int N_, int FAMS_>
struct SepGeo {
  static constexpr int N = N_, K = N * N, FAMS = FAMS_;
  static constexpr int NFAM = FAMS == 3 ? 2 : 1;
  static constexpr int M = NFAM * K;
  static constexpr int WPN = N == 64 ? 4 : 1;          // waves per node
  static constexpr int NPG = 4 / WPN;                  // nodes per workgroup
  static constexpr int TT = N / 16;                    // 16-wide tiles of a side
  static constexpr int TQ = TT / WPN;                  // q tiles per wave
  static constexpr int VPL = NFAM * 16;                // correlations per lane: 4 TQ TT of each family
  static constexpr int PW = N / 8, PH = N / 8;         // patch of a lane over the node's waves
  static constexpr int RPW = PH / WPN;                 // patch rows held by one wave
  static constexpr int KS = N / 32;                    // k-steps (32) of a product
  // LDS rows of the residual, padded by 16 bytes: 16 consecutive rows read
  // at one column offset (16 bytes per lane) fall on all banks once.
  static constexpr int ROWB = 2 * N + 16;
  static constexpr int HALFB = N * ROWB;               // hi rows, then lo rows
  static constexpr int RBYTES = 2 * HALFB;
  static_assert(RBYTES >= 4 * K, "the gather stages FP32 pixels in the residual buffer");
  // Power of two on the DCT operands (and on the Haar magnitudes): their
  // FP16 remainders are then normal numbers.
  static constexpr float TS = 128.f;
  static_assert(4 * TQ * TT == 16 && VPL <= 32, "one vector per family, one mask word per lane");
  // Table operands, 16 bytes at a time: values of each family, then the DCT
  // remainders; then the signs of the Haar table (bytes) and FP32 <T_0[p],
  // T_1[p']> with its transpose.
  static constexpr int NOPS = FAMS == 3 ? 3 : (FAMS == AQMP_HAAR ? 1 : 2);
  static constexpr int EOPS = NOPS * TT * KS * 64;
  static constexpr int SGNB = FAMS == AQMP_DCT ? 0 : K;   // bytes of signs
  static constexpr size_t OFF_S = EOPS, OFF_X = OFF_S + SGNB / 16;
  static constexpr size_t BYTES = 16 * OFF_X + (NFAM == 2 ? 8 * (size_t)K : 0);
  static constexpr bool XLDS = NFAM == 2 && N == 32;     // that table in LDS (N = 64: 32 KB, no room beside a second workgroup)
};

// Whether family f of a dictionary is the Haar one.
template <class G>
__device__ constexpr bool sep_haar(int f) { return G::FAMS == AQMP_HAAR || (G::FAMS == 3 && f == 1); }

// Two FP32 values -> packed FP16 halves and their packed remainders.  The
// mixed-precision FMA takes FP16 sources and rounds its result to FP16 in
// place, so a value costs one and a half instructions here (BF16 needs
// three: no such FMA exists for it).  op_sel_hi marks an FP16 source, op_sel
// its upper half.  The remainders are matrix-core operands: two wait states
// after their last write, which the compiler does not add behind inline
// assembly.
__device__ inline void sp_split2(float a, float b, uint32_t& h, uint32_t& l) {
  const auto p = __builtin_amdgcn_cvt_pkrtz(a, b);
  __builtin_memcpy(&h, &p, 4);
  __asm__("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(l) : "v"(h), "v"(a));
  __asm__("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\ts_nop 1" : "+v"(l) : "v"(h), "v"(b));
}
// The same for a * s and b * s (s a power of two).
__device__ inline void sp_split2_scaled(float a, float b, float s, uint32_t& h, uint32_t& l) {
  __asm__("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(a), "v"(s));
  __asm__("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(b), "v"(s));
  __asm__("v_fma_mixlo_f16 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(l) : "v"(a), "v"(s), "v"(h));
  __asm__("v_fma_mixhi_f16 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(l) : "v"(b), "v"(s), "v"(h));
}

// Writes the operands of one dictionary level (see SepGeo), made once with
// the dictionary: word ((o TT + t) KS + ks) 64 + lane holds T[16 t + m][x] at
// the eight pixels x of k-slots (ks, g, 0..7).  A Haar row is one magnitude
// times -1, 0 or 1: its operands are those signs, exact in FP16 (no remainder,
// two products instead of three), and the magnitudes of the row and the
// column multiply the finished correlation.  xg: FP64 <T_0[p], T_1[p']>.
template <class G>
__device__ inline void sep_make_ops(const double* __restrict__ tab, const double* __restrict__ xg,
                                    uint4* __restrict__ out) {
  constexpr int N = G::N;
  const int tid = threadIdx.x;
  for (int i = tid; i < G::EOPS; i += 256) {
    const int lane = i & 63, m = lane & 15, g = lane >> 4;
    const int ks = (i >> 6) % G::KS, t = (i >> 6) / G::KS % G::TT, o = (i >> 6) / (G::KS * G::TT);
    const int f = o < G::NFAM ? o : 0;
    const bool haar = sep_haar<G>(f);
    const double* row = tab + (size_t)f * G::K + (16 * t + m) * N;
    sp_h8 v;
    for (int j = 0; j < 8; ++j) {
      const double d = row[32 * ks + 16 * (j >> 2) + 4 * g + (j & 3)];
      const float w = haar ? (d > 0.0 ? 1.f : (d < 0.0 ? -1.f : 0.f)) : (float)d * G::TS;
      const _Float16 h = (_Float16)w;
      v[j] = o < G::NFAM ? h : (_Float16)(w - (float)h);
    }
    __builtin_memcpy(&out[i], &v, 16);
  }
  if constexpr (G::SGNB > 0) {
    const double* h = tab + (G::FAMS == 3 ? G::K : 0);
    int8_t* sg = (int8_t*)(out + G::OFF_S);
    for (int i = tid; i < G::K; i += 256) sg[i] = h[i] > 0.0 ? 1 : (h[i] < 0.0 ? -1 : 0);
  }
  if constexpr (G::NFAM == 2) {
    float* x = (float*)(out + G::OFF_X);
    for (int i = tid; i < G::K; i += 256) {
      x[i] = (float)xg[i];
      x[G::K + i] = (float)xg[(i % N) * N + i / N];
    }
  }
}

template <int N, int FAMS>
__global__ __launch_bounds__(256) void k_sep_ops(const double* __restrict__ tab, const double* __restrict__ xg,
                                                 uint4* __restrict__ out) {
  sep_make_ops<SepGeo<N, FAMS>>(tab, xg, out);
}

// All correlations of the residual in sR with the wave's columns q:
// C[f][4 (i TT + tp) + r] = c of atom (f, p = 16 tp + 4 g + r, q = 16 (TQ wq + i) + m).
// ops: the table operands in LDS (in registers they would fill half of those
// of the steps between two calls; from memory a call took 12 000 to 45 000
// cycles, every workgroup reading the same lines).
template <class G>
__device__ inline void sep_correlate(const char* sR, const uint4* ops, int wq, const float (&mq)[G::TQ], const float (&mp0)[4],
                                     const float (&mp)[G::TT], sp_f32x16 (&C)[G::NFAM]) {
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  auto op = [&](int o, int t, int ks) -> sp_h8 { return *(const sp_h8*)&ops[((o * G::TT + t) * G::KS + ks) * 64 + lane]; };
  const char* base = sR + m * G::ROWB + 16 * g;
#pragma unroll
  for (int f = 0; f < G::NFAM; ++f) {
    constexpr int L = G::NOPS - 1;                       // the DCT's remainders
    const bool haar = sep_haar<G>(f);                    // no remainders
    sp_f32x4 D[G::TQ][G::TT], c[G::TQ][G::TT];
#pragma unroll
    for (int i = 0; i < G::TQ; ++i)
#pragma unroll
      for (int t = 0; t < G::TT; ++t) D[i][t] = c[i][t] = sp_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) {
      sp_h8 a[G::TQ], al[G::TQ];
#pragma unroll
      for (int i = 0; i < G::TQ; ++i) {
        a[i] = op(f, wq * G::TQ + i, ks);
        if (!haar) al[i] = op(L, wq * G::TQ + i, ks);
      }
#pragma unroll
      for (int ty = 0; ty < G::TT; ++ty) {
        const sp_h8 rh = *(const sp_h8*)(base + 16 * ty * G::ROWB + 64 * ks);
        const sp_h8 rl = *(const sp_h8*)(base + G::HALFB + 16 * ty * G::ROWB + 64 * ks);
#pragma unroll
        for (int i = 0; i < G::TQ; ++i) {
          D[i][ty] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rh, a[i], D[i][ty], 0, 0, 0);
          if (!haar) D[i][ty] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rh, al[i], D[i][ty], 0, 0, 0);
          D[i][ty] = __builtin_amdgcn_mfma_f32_16x16x32_f16(rl, a[i], D[i][ty], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int ks = 0; ks < G::KS; ++ks) {
      sp_h8 zh[G::TQ], zl[G::TQ];
#pragma unroll
      for (int i = 0; i < G::TQ; ++i) {
        uint32_t h[4], l[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const sp_f32x4& d = D[i][2 * ks + (j >> 1)];
          sp_split2(d[2 * (j & 1)], d[2 * (j & 1) + 1], h[j], l[j]);
        }
        __builtin_memcpy(&zh[i], h, 16);
        __builtin_memcpy(&zl[i], l, 16);
      }
#pragma unroll
      for (int tp = 0; tp < G::TT; ++tp) {
        const sp_h8 b = op(f, tp, ks);
        sp_h8 bl;
        if (!haar) bl = op(L, tp, ks);
#pragma unroll
        for (int i = 0; i < G::TQ; ++i) {
          c[i][tp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b, zh[i], c[i][tp], 0, 0, 0);
          if (!haar) c[i][tp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bl, zh[i], c[i][tp], 0, 0, 0);
          c[i][tp] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b, zl[i], c[i][tp], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int i = j / (4 * G::TT), tp = (j >> 2) % G::TT, r = j & 3;
      C[f][j] = haar ? c[i][tp][r] * ((tp == 0 ? mp0[r] : mp[tp]) * mq[i]) : c[i][tp][r];
    }
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

// Tables in LDS: operands of the correlation; FP64 1D rows, the DCT as it
// is, a Haar row one magnitude times -1, 0 or 1 (exact products), kept as
// signs and one FP64 magnitude per scale (row 0, then rows [2^j, 2^(j+1))).
template <class G>
struct SepTab {
  uint4 ops[G::EOPS];
  double dct[(G::FAMS & AQMP_DCT) ? G::K + 2 * G::N : 1];   // rows N, N + 1: ones and 1/N, of the constant atom
  uint4 sgn[G::SGNB ? G::SGNB / 16 : 1];
  float x[G::XLDS ? 2 * G::K : 1];
  double mag[8];
};

__device__ inline int sep_haar_scale(int p) { return p == 0 ? 0 : 32 - __builtin_clz((unsigned)p); }

template <class G>
__device__ inline void sep_load_tab(SepTab<G>& S, const double* __restrict__ tab, const uint4* __restrict__ ops) {
  const int tid = threadIdx.x;
#pragma unroll 6
  for (int i = tid; i < G::EOPS; i += 256) S.ops[i] = ops[i];
  if constexpr ((G::FAMS & AQMP_DCT) != 0) {
#pragma unroll 8
    for (int i = tid; i < G::K / 2; i += 256) ((double2*)S.dct)[i] = ((const double2*)tab)[i];
    if (tid < 2 * G::N) S.dct[G::K + tid] = tid < G::N ? 1.0 : 1.0 / G::N;
  }
  if constexpr (G::SGNB > 0) {
    for (int i = tid; i < G::SGNB / 16; i += 256) S.sgn[i] = ops[G::OFF_S + i];
    // the first row of a scale starts at pixel 0
    const double* h = tab + (G::FAMS == 3 ? G::K : 0);
    if (tid < 8) {
      const int row = tid == 0 ? 0 : 1 << (tid - 1);
      S.mag[tid] = row < G::N ? h[row * G::N] : 0.0;
    }
  }
  if constexpr (G::XLDS)
    for (int i = tid; i < G::K / 2; i += 256) ((uint4*)S.x)[i] = ops[G::OFF_X + i];
}

// The FP64 factors of atom `at` (uniform) over the lane's patch: tq at its
// columns px.., tp at its rows py.. of the whole node's patch, ty at those of
// its wave's rows.  The constant atom is 1/N times ones.
template <class G>
__device__ inline void sep_factors(const SepTab<G>& S, int at, int px, int py, int wq, double (&tq)[G::PW],
                                   double (&tp)[G::PH], double (&ty)[G::RPW]) {
  constexpr int N = G::N, K = G::K, PW = G::PW, PH = G::PH, RPW = G::RPW;
  const int f = at / K, q = (at % K) / N, p = at % N;
  const bool dc = p == 0 && q == 0;
  if (G::FAMS == AQMP_HAAR || (G::FAMS == 3 && f == 1)) {
    if constexpr ((G::FAMS & AQMP_HAAR) != 0) {
      const double mg = G::FAMS == AQMP_HAAR && dc ? 1.0 : S.mag[sep_haar_scale(q)];
      const double mh = G::FAMS == AQMP_HAAR && dc ? 1.0 / N : S.mag[sep_haar_scale(p)];
      uint32_t w[PW / 4], v[PH / 4];
      __builtin_memcpy(w, __builtin_assume_aligned((const char*)S.sgn + q * N + px, PW), PW);
      __builtin_memcpy(v, __builtin_assume_aligned((const char*)S.sgn + p * N + py, PH), PH);
#pragma unroll
      for (int j = 0; j < PW; ++j) tq[j] = (double)((int32_t)(w[j / 4] << (24 - 8 * (j % 4))) >> 24) * mg;
#pragma unroll
      for (int i = 0; i < PH; ++i) tp[i] = (double)((int32_t)(v[i / 4] << (24 - 8 * (i % 4))) >> 24) * mh;
      if constexpr (G::WPN > 1) {
        uint16_t u;
        __builtin_memcpy(&u, __builtin_assume_aligned((const char*)S.sgn + p * N + py + wq * RPW, 2), 2);
#pragma unroll
        for (int i = 0; i < RPW; ++i) ty[i] = (double)((int32_t)((uint32_t)u << (24 - 8 * i)) >> 24) * mh;
      }
    }
  } else {
    if constexpr ((G::FAMS & AQMP_DCT) != 0) {
      const double* rq = S.dct + (dc ? N : q) * N + px;
      const double* rp = S.dct + (dc ? N + 1 : p) * N + py;
#pragma unroll
      for (int j = 0; j < PW; ++j) tq[j] = rq[j];
#pragma unroll
      for (int i = 0; i < PH; ++i) tp[i] = rp[i];
      if constexpr (G::WPN > 1) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) ty[i] = rp[wq * RPW + i];
      }
    }
  }
  if constexpr (G::WPN == 1) {
#pragma unroll
    for (int i = 0; i < RPW; ++i) ty[i] = tp[i];
  }
}

__device__ inline double sep_bcast_f64(double d) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(d);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)u);
  const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The arg-max over the tiles of the wave's columns q that hold a candidate (mask,
// see k_pursuit_sep) of the correlations in FP64, made anew from the FP32
// residual in sr (rows of N + 4): the products of sep_correlate on the FP64
// matrix cores, whose layouts fit each other the same way.  (The Haar rows from
// N / 2 on are of two pixels: 16 of them, of 32.)
template <class G>
__device__ inline LaneBest sep_exact(const float* sr, const SepTab<G>& S, int wq, uint32_t mask, double w) {
  constexpr int N = G::N, K = G::K, TT = G::TT, TQ = G::TQ;
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  uint32_t tiles = 0u;
#pragma unroll
  for (int k = 0; k < G::VPL / 4; ++k) tiles |= __ballot((mask >> (G::VPL - 4 - 4 * k)) & 15u) != 0ull ? 1u << k : 0u;
  LaneBest best;
#pragma unroll 1
  for (int f = 0; f < G::NFAM; ++f) {
    const bool haar = sep_haar<G>(f);
    auto table = [&](int row, int col) -> double {
      if (haar) return (double)((const int8_t*)S.sgn)[row * N + col] * S.mag[sep_haar_scale(row)];
      return S.dct[(G::FAMS & AQMP_DCT) ? row * N + col : 0];
    };
#pragma unroll 1
    for (int i = 0; i < TQ; ++i) {
      const uint32_t row = (tiles >> (4 * f + TT * i)) & ((1u << TT) - 1u);
      if (row == 0u) continue;
      const int tq = wq * TQ + i, q = 16 * tq + m;
      d4 D[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) D[t] = d4{0.0, 0.0, 0.0, 0.0};
      const int x0 = haar && 2 * tq >= TT ? 32 * tq - N : 0, x1 = haar && 2 * tq >= TT ? x0 + 32 : N;
#pragma unroll 1
      for (int x = x0; x < x1; x += 8) {
#pragma unroll
        for (int j = 0; j < 8; j += 4) {
          const double b = table(q, x + j + g);
#pragma unroll
          for (int t = 0; t < TT; ++t) D[t] = mfma64((double)sr[(16 * t + m) * (N + 4) + x + j + g], b, D[t]);
        }
      }
#pragma unroll 1
      for (int tp = 0; tp < TT; ++tp) {
        if (!((row >> tp) & 1u)) continue;
        d4 c = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int y = 0; y < N; y += 4) c = mfma64(table(16 * tp + m, y + g), D[y / 16][y / 4 % 4], c);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int at = f * K + q * N + 16 * tp + g + 4 * r;
          best.take(f == 1 && at == K ? 0.0 : c[r], at, w);   // (the second constant atom)
        }
      }
    }
  }
  best.over_wave(w);
  return best;
}

// Candidates are re-scored one after the other.  Where more lanes than this hold
// one, all of their tiles are made in FP64 instead (sep_exact, up to 12 000 cycles
// a family at N = 64 against 1 000 per candidate); atoms within 2^-42 ||r|| of the
// largest tie, that is by all but the rounding of those sums, and the lowest is
// taken.  In the Haar basis alone a dithered or a checkered plane ties 200 to
// 1 024 atoms at every step: 256 x 256 checkered, 16 steps, N = 64 / 32: 129 / 81
// us, with all of them re-scored 7 772 / 1 384, eight per step in launches of
// their own 709 / 321.
constexpr int kSepMany = 12;

// Workgroups per CU: as many as fit the registers without sep_exact (and LDS).
template <int N, int FAMS>
__global__ __launch_bounds__(256, N == 64 ? (FAMS == 2 ? 3 : 2) : (FAMS == 3 ? 3 : 4)) void k_pursuit_sep(const JobDev* __restrict__ jobs, LevelDev lv,
                                                        const int32_t* __restrict__ count_ptr,
                                                        int32_t* __restrict__ queue, int32_t lg,
                                                        const double* __restrict__ tab,
                                                        const uint4* __restrict__ ops) {
  using G = SepGeo<N, FAMS>;
  constexpr int K = G::K, WPN = G::WPN, NPG = G::NPG, PW = G::PW, PH = G::PH, RPW = G::RPW, VPL = G::VPL;
  // Per node: operand rows of the residual; the gather's pixels; N = 64: row
  // sums that the waves exchange and their masks (in turn, barriers between).
  __shared__ __attribute__((aligned(16))) char sRes[NPG][G::RBYTES];
  __shared__ __attribute__((aligned(16))) SepTab<G> sTab;
  __shared__ __attribute__((aligned(16))) uint4 sTop[2];   // per wave: largest |c|; its atom, with the top bit if there are others
  __shared__ double sRed[4], sBest[4];
  __shared__ int sNode[4], sBestAt[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = WPN > 1 ? wv : 0;                       // wave within the node
  const int grp = WPN > 1 ? 0 : wv;                      // node slot of the workgroup
  char* sR = sRes[grp];
  double(*sPart)[PH][64] = (double(*)[PH][64])sR;        // two buffers, WPN > 1
  uint32_t* sMask = (uint32_t*)(sR + 2 * sizeof(*sPart));
  static_assert(WPN == 1 || 2 * sizeof(*sPart) + 1024 <= G::RBYTES, "exchange buffers");
  static_assert(4 * N * (N + 4) <= G::RBYTES, "FP32 pixels for sep_exact");
  // [f][p][p']: row p of family f against the other family
  const float* gram = G::XLDS ? sTab.x : (const float*)(ops + G::OFF_X);
  sep_load_tab<G>(sTab, tab, ops);
  // Haar magnitudes of the lane's columns and rows: a row's is its value at
  // the first pixel of its support
  float mq[G::TQ] = {}, mp0[4] = {}, mp[G::TT] = {};
  if constexpr (G::FAMS != AQMP_DCT) {
    const double* h = tab + (G::FAMS == 3 ? K : 0);
    auto mag = [&](int row) -> float {
      const int top = row > 0 ? 1 << (31 - __builtin_clz((unsigned)row)) : N;
      return (float)h[row * N + (row > 0 ? (row - top) * (N / top) : 0)];
    };
#pragma unroll
    for (int i = 0; i < G::TQ; ++i) mq[i] = mag(16 * (wq * G::TQ + i) + (lane & 15)) * (G::TS * G::TS);
#pragma unroll
    for (int r = 0; r < 4; ++r) mp0[r] = mag(4 * (lane >> 4) + r);
#pragma unroll
    for (int tp = 1; tp < G::TT; ++tp) mp[tp] = mag(16 * tp);   // one scale from row 16 up to the next power of two
  }
  __syncthreads();
  const int count = *count_ptr;
  const int py = (lane >> 3) * PH + wq * RPW;            // first pixel of the lane's rows
  const int px = (lane & 7) * PW;
  // The first nodes are dealt out in order, the others by the queues: queue
  // k holds every kQueues-th node after the first ones.
  const int q0 = (int)gridDim.x * NPG;
  int qk = (int)blockIdx.x % kQueues;
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
        ep = wave_sum_f64(ep);                           // group_sum<256>'s order
        if (lane == 0) sRed[wv] = ep;
        sep_sync<WPN>();
        e = (sRed[0] + sRed[1]) + (sRed[2] + sRed[3]);
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
          ev[vw] = wave_sum_f64(ev[vw]);
        }
        e = (ev[0] + ev[1]) + (ev[2] + ev[3]);
      }
    }
    e = sep_bcast_f64(e);
    if constexpr (WPN == 1) sep_sync<WPN>();
    double r[RPW][PW];                                   // FP32 values
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int j = 0; j < PW; ++j) r[i][j] = (double)((const float*)sR)[(py + i) * N + px + j];
    sep_sync<WPN>();
    // Scale 2^-sh of the operand rows: ||r|| goes to [2^7, 2^8), so that the
    // first product (at most 2^15) and the remainders stay inside FP16's
    // range.  The norm of FP32 pixels can lie beyond FP32's range: what is
    // past 120 of sh, either way, goes to the pixels in FP64.
    auto scale_of = [](double en) -> int {
      const int ex = (int)((unsigned long long)__double_as_longlong(en) >> 52) - 1023;
      return (ex >> 1) - 7;
    };
    auto pow2 = [](int x) -> double { return __longlong_as_double((long long)(1023 + x) << 52); };
    auto put_rows = [&](int sh) {                        // the lane's pixels into the operand rows
      const int s0 = sh < -120 ? -120 : (sh > 120 ? 120 : sh);
      const float sc = __uint_as_float((uint32_t)(127 - s0) << 23);
      const double over = pow2(s0 - sh);                 // 1 but beyond FP32's range
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        char* row = sR + (py + i) * G::ROWB;
        uint32_t h[PW / 2], l[PW / 2];
        float v[PW];
#pragma unroll
        for (int j = 0; j < PW; ++j) v[j] = (float)(r[i][j] * over);
#pragma unroll
        for (int j = 0; j < PW / 2; ++j) sp_split2_scaled(v[2 * j], v[2 * j + 1], sc, h[j], l[j]);
        // in the order of the k-slots: pixel x is value 4 ((x / 16) % 2) + x % 4
        // of the slots (x / 32, (x / 4) % 4)
#pragma unroll
        for (int j = 0; j < PW; j += 4) {
          char* at = row + 2 * (32 * (px >> 5) + 8 * ((px >> 2) & 3) + 4 * ((px >> 4) & 1) + 2 * j);
          *(uint2*)at = make_uint2(h[j / 2], h[j / 2 + 1]);
          *(uint2*)(at + G::HALFB) = make_uint2(l[j / 2], l[j / 2 + 1]);
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
    sp_f32x16 C[G::NFAM];                                // correlations, times gain
    float win = 0.f, mx = 0.f;
    uint32_t mask = 0u;                                  // bit VPL - 1 - j: value j is within win of the wave's largest
    uint32_t best = 0u;                                  // the wave's candidate, with the top bit if there are others or none
    auto atom_of = [&](int w, int l, int bit) -> int {   // wave of the node, lane, bit of its mask
      const int j = VPL - 1 - bit, f = j >> 4, i = (j & 15) / (4 * G::TT), tp = (j >> 2) % G::TT;
      return f * K + (16 * (w * G::TQ + i) + (l & 15)) * N + 16 * tp + 4 * (l >> 4) + (j & 3);
    };
    // The wave's largest |c| and its atoms within the window, to the node's
    // other waves.
    auto top = [&]() {
      if constexpr (G::NFAM == 2) {
        // the second family's constant atom equals the first's, which wins the tie
        if (wq == 0 && lane == 0) C[1][0] = 0.f;
      }
      auto val = [&](int j) -> float { return C[j >> 4][j & 15]; };
      float m0 = 0.f, m1 = 0.f;
#pragma unroll
      for (int j = 0; j < VPL; j += 4) {
        m0 = fmaxf(fmaxf(fabsf(val(j)), fabsf(val(j + 1))), m0);
        m1 = fmaxf(fmaxf(fabsf(val(j + 2)), fabsf(val(j + 3))), m1);
      }
      mx = wave_max_f32(fmaxf(m0, m1));
      // the sign of thr - |c| into the mask: two instructions per value
      const float thr = mx - win;
      mask = 0u;
#pragma unroll
      for (int j = 0; j < VPL; ++j)
        mask = __builtin_amdgcn_alignbit(mask, __float_as_uint(thr - fabsf(val(j))), 31);
      if (!(mx > 0.f && mx < __builtin_inff())) mask = 0u;   // undefined sums: nothing to compare
      const unsigned long long near = __ballot(mask != 0u);
      const bool others = __popcll(near) != 1 || __ballot((mask & (mask - 1u)) != 0u) != 0ull;
      const int l = near ? __builtin_ctzll(near) : 0;
      const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)mask, l);
      best = (uint32_t)atom_of(wq, l, bits ? __builtin_ctz(bits) : 0) | (others ? 0x80000000u : 0u);
      if constexpr (WPN > 1)
        if (lane == 0) {
          ((uint32_t*)sTop)[wv] = __float_as_uint(mx);
          ((uint32_t*)sTop)[4 + wv] = best;
        }
    };
    int given = -1;                                      // the step's atom, where it was taken among many
    while (st == ST_RUN) {
      if (!(e > 0.0 && e < __builtin_inf())) {           // a zero residual, or undefined pixels: nothing to select
        st = ST_ZERO;
        break;
      }
      // ---- correlations from the residual ----
      const int sh = scale_of(e);
      sep_sync<WPN>();                                   // the sums of the last step are read
      put_rows(sh);
      sep_sync<WPN>();
      sep_correlate<G>(sR, sTab.ops, wq, mq, mp0, mp, C);
      const double gain = pow2(-sh) * (double)(G::TS * G::TS);
      win = __builtin_amdgcn_sqrtf((float)(e * pow2(-sh) * pow2(-sh))) * (1.0001f * 0x1p-13f * G::TS * G::TS);
      top();
      sep_sync<WPN>();
      // They hold while ||r|| is at least half of what it is now, for at most
      // 64 steps (and to the end of a window of records).
      const double elim = fmax(eps2, 0.25 * e), emax = 4.0 * e;
      const int tlim = min(kmax, (t & ~63) + 64);
      bool many = false;
      for (;;) {
        uint32_t pick = best;
        if constexpr (WPN > 1) {
          const uint4 a = sTop[0], b = sTop[1];
          const float wm[4] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w)};
          const uint32_t wb[4] = {b.x, b.y, b.z, b.w};
          mx = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
          const float thr = mx - win;
          uint32_t n = 0u;
          pick = 0u;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            pick = wm[w] >= thr ? wb[w] : pick;
            n += wm[w] >= thr ? 1u : 0u;
          }
          pick = n == 1u ? pick : 0x80000000u;
        }
        pick = (uint32_t)__builtin_amdgcn_readfirstlane((int)pick);
        if (given >= 0) pick = (uint32_t)given;
        given = -1;
        // rows of the 1D Gram matrix for the update of the correlations (read
        // ahead of the re-score that hides them)
        sp_f32x4 gp[G::NFAM == 2 ? G::TT : 1];
        float gq[G::NFAM == 2 ? G::TQ : 1];
        auto gram_rows = [&](int at) {
          if constexpr (G::NFAM == 2) {
            const int f = at / K, q = (at % K) / N, p = at % N;
            const float* x = gram + (size_t)f * K;
#pragma unroll
            for (int tp = 0; tp < G::TT; ++tp) gp[tp] = *(const sp_f32x4*)(x + p * N + 16 * tp + 4 * (lane >> 4));
#pragma unroll
            for (int i = 0; i < G::TQ; ++i) gq[i] = x[q * N + 16 * (wq * G::TQ + i) + (lane & 15)];
          }
        };
        // (Branches are marked with the way most steps go, whose code then lies in
        // one piece: three 2048 x 2048 planes 563 -> 559 us.)
        // ---- FP64 re-score (k_select's patches and order of operations) ----
        double tq[PW], tp8[PH], ty[RPW];
        auto rescore = [&](int at) -> double {
          sep_factors<G>(sTab, at, px, (lane >> 3) * PH, wq, tq, tp8, ty);
          double all[PH], sr[RPW];
#pragma unroll
          for (int i = 0; i < RPW; ++i) {
            sr[i] = 0.0;
#pragma unroll
            for (int j = 0; j < PW; ++j) sr[i] = fma(r[i][j], tq[j], sr[i]);
          }
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
#pragma unroll
          for (int i = 0; i < PH; ++i) part = fma(tp8[i], all[i], part);
          return wave_sum_f64(part);
        };
        int atom = -1;
        double coef = 0.0, mag = -1.0;
        if (__builtin_expect(!(pick >> 31), 1)) {
          gram_rows((int)pick);
          coef = rescore((int)pick);
          mag = fabs(coef);
          atom = (int)pick;
        } else if (mx < __builtin_inff()) {
          // several atoms within the window: every one of them, lowest index on
          // ties (a wave's mask is relative to its own largest: no fewer atoms)
          if constexpr (WPN > 1) {
            // a wave whose largest is outside the node's window has no candidate
            mask = __uint_as_float(((const uint32_t*)sTop)[wq]) >= mx - win ? mask : 0u;
          }
          int held[WPN], n = 0;                          // lanes of each wave with a candidate
          held[0] = __popcll(__ballot(mask != 0u));
          if constexpr (WPN > 1) {
            sMask[tid] = mask;
            if (lane == 0) sBestAt[wv] = held[0];
            sep_sync<WPN>();
#pragma unroll
            for (int w = 0; w < WPN; ++w) held[w] = __builtin_amdgcn_readfirstlane(sBestAt[w]);
          }
#pragma unroll
          for (int w = 0; w < WPN; ++w) n += held[w];
          if (__builtin_expect(n > kSepMany, 0)) {
            many = true;
            break;
          }
          for (int w = 0; w < WPN; ++w) {
            if (held[w] == 0) continue;
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
            gram_rows(atom);
            sep_factors<G>(sTab, atom, px, (lane >> 3) * PH, wq, tq, tp8, ty);
          }
        }
        if (atom < 0 || mag == 0.0) {
          st = ST_ZERO;
          break;
        }
        // ---- rank-1 update, norm, record, stop test ----
        double eh[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
          eh[i] = 0.0;
#pragma unroll
          for (int j = 0; j < PW; ++j) {
            const double phi = ty[i] * tq[j];
            const double rn = (double)(float)fma(-coef, phi, r[i][j]);
            r[i][j] = rn;
            eh[i] = fma(rn, rn, eh[i]);
          }
        }
        if constexpr (WPN > 1) {
#pragma unroll
          for (int i = 0; i < RPW; ++i) sPart[par][wq * RPW + i][lane] = eh[i];
        }
        // ---- correlations of the new residual: the atom's own loses its
        // coefficient, its family's others are orthogonal to it, those of the
        // other family lose <phi, phi'> = X[p][p'] X[q][q'] times it ----
        {
          const int f = atom / K, q = (atom % K) / N, p = atom % N;
          const float cs = (float)(coef * gain);
          const float own = lane == (((p & 15) >> 2) << 4 | (q & 15)) && (WPN == 1 || (q >> 4) / G::TQ == wq) ? cs : 0.f;
          const int j = (((q >> 4) % G::TQ) * G::TT + (p >> 4)) * 4 + (p & 3);
          // (no branch on the family, whose joins copied all of them: the atom's
          // own family takes zero times the products)
          if constexpr (G::NFAM == 2) {
#pragma unroll
            for (int f2 = 0; f2 < 2; ++f2)
#pragma unroll
              for (int i = 0; i < G::TQ; ++i) {
                const float s = f2 != f ? -(cs * gq[i]) : 0.f;
#pragma unroll
                for (int x = 0; x < 4 * G::TT; ++x)
                  C[f2][i * 4 * G::TT + x] = fmaf(s, gp[x >> 2][x & 3], C[f2][i * 4 * G::TT + x]);
              }
          }
#pragma unroll
          for (int f2 = 0; f2 < G::NFAM; ++f2) C[f2][j] -= f2 == f ? own : 0.f;
        }
        top();
        double ew = 0.0;
        if constexpr (WPN > 1) {
          sep_sync<WPN>();
#pragma unroll
          for (int i = 0; i < PH; ++i) ew += sPart[par][i][lane];
          par ^= 1;
        } else {
#pragma unroll
          for (int i = 0; i < PH; ++i) ew += eh[i];
        }
        e = wave_sum_f64(ew);
        if (lane == (t & 63)) {
          rec_i = atom;
          rec_c = coef;
        }
        ++t;
        if (!(e >= elim && e < emax && t < tlim)) break;
      }
      if (__builtin_expect(many, 0)) {
        sep_sync<WPN>();                                 // the masks are read
        float* sr = (float*)sR;
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
          for (int j = 0; j < PW; ++j) sr[(py + i) * (N + 4) + px + j] = (float)r[i][j];
        sep_sync<WPN>();
        const double w = 0x1p-42 * __builtin_sqrt(e);
        const LaneBest found = sep_exact<G>(sr, sTab, wq, mask, w);
        given = found.atom;
        if constexpr (WPN > 1) {
          if (lane == 0) {
            sBest[wv] = found.mag;
            sBestAt[wv] = found.atom;
          }
          sep_sync<WPN>();
          const double mag = fmax(fmax(sBest[0], sBest[1]), fmax(sBest[2], sBest[3]));
          given = 0x7fffffff;
          for (int v = 0; v < 4; ++v) given = sBest[v] >= mag - w ? min(given, sBestAt[v]) : given;
        }
        given = __builtin_amdgcn_readfirstlane(given);
        continue;
      }
      if (st != ST_RUN) break;
      if ((t & 63) == 0 && wq == 0) {
        lv.rec_idx[rec0 + t - 64 + lane] = rec_i;
        lv.rec_coef[rec0 + t - 64 + lane] = rec_c;
      }
      if (e < eps2)
        st = ST_ACC;
      else if (t >= kmax)
        st = ST_SPARSE;
    }
    // The next node, not before this one is done: nodes differ in length by
    // the whole pursuit (taken with this node's gather, N = 64 took 277 instead
    // of 243 us on three 2048 x 2048 planes, N = 32 106 instead of 86).  N = 64
    // also empties the other queues (search round 575 -> 549 us); with a node
    // per wave or slot the look at them costs more than it evens out.
    int ahead = 0;
    if constexpr (WPN > 1) {
      if (tid == 0) ahead = next_node(queue, qk, q0, count);
    } else {
      if (lane == 0) ahead = q0 + atomicAdd(queue + qk * kQueuePad, 1) * kQueues + qk;
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
    if (WPN > 1 ? tid == 0 : lane == 0) sNode[grp] = ahead;
    sep_sync<WPN>();
    node = __builtin_amdgcn_readfirstlane(sNode[grp]);
    sep_sync<WPN>();
  }
}

template <int N, int FAMS>
hipError_t launch_sep_n(const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue, int64_t cap,
                        const double* tab, const void* ops, hipStream_t s) {
  using G = SepGeo<N, FAMS>;
  // Nodes come from a counter, so the grid is as many workgroups as are
  // resident at once (at most one per NPG nodes of the level).
  int dev = 0, n_cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pursuit_sep<N, FAMS>, 256, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  int64_t wgs = (cap + G::NPG - 1) / G::NPG;
  if (wgs > (int64_t)n_cus * per_cu) wgs = (int64_t)n_cus * per_cu;
  if (wgs < 1) wgs = 1;
  hipLaunchKernelGGL((k_pursuit_sep<N, FAMS>), dim3((unsigned)wgs), dim3(256), 0, s, jobs, lv, count, queue,
                     ilog2(N), tab, (const uint4*)ops);
  return hipGetLastError();
}

template <int N, int FAMS>
hipError_t launch_sep_ops_n(const double* tab, const double* xg, void* out, hipStream_t s) {
  hipLaunchKernelGGL((k_sep_ops<N, FAMS>), dim3(1), dim3(256), 0, s, tab, xg, (uint4*)out);
  return hipGetLastError();
}

}  // namespace

// Runs CALL with NN, FF set for a block size and family mask.
#define AQMP_SEP_F(NN_, CALL)                   \
  {                                             \
    constexpr int NN = NN_;                     \
    switch (families) {                         \
      case 1: { constexpr int FF = 1; CALL; }   \
      case 2: { constexpr int FF = 2; CALL; }   \
      case 3: { constexpr int FF = 3; CALL; }   \
    }                                           \
  }
#define AQMP_SEP(CALL)                   \
  switch (n) {                           \
    case 32: AQMP_SEP_F(32, CALL) break; \
    case 64: AQMP_SEP_F(64, CALL) break; \
  }

size_t sep_ops_bytes(int n, uint32_t families) {
  AQMP_SEP(return (SepGeo<NN, FF>::BYTES))
  return 0;
}

hipError_t launch_sep_ops(int n, uint32_t families, const double* tab, const double* xg, void* out, hipStream_t s) {
  AQMP_SEP(return (launch_sep_ops_n<NN, FF>(tab, xg, out, s)))
  return hipErrorInvalidValue;
}

hipError_t launch_pursuit_sep(int n, uint32_t families, const JobDev* jobs, LevelDev lv, const int32_t* count,
                              int32_t* queue, int64_t cap, const double* tab, const void* ops, hipStream_t s) {
  AQMP_SEP(return (launch_sep_n<NN, FF>(jobs, lv, count, queue, cap, tab, ops, s)))
  return hipErrorInvalidValue;
}

}  // namespace aqmp
