// kernels_sub.hip - whole-level Matching Pursuit of the dense solver for small
// blocks on the matrix cores: N = 8 and 16.  A wave runs several nodes side by
// side (slots of LPS lanes), with no workgroup barrier; the residual stays in
// registers from the gather to the last step.
//
// The correlation is the factored one of kernels_sep.hip: C_f = T_f R T_f^T
// for every family f, first D1[y][q] = sum_x R[y][x] T[q][x], then C[p][q] =
// sum_y T[p][y] D1[y][q], whose lane layout makes D1 the B operand of the
// second product as it is, and with FP16 halves: the value and its remainder
// of one operand sit side by side in the 32-deep contraction of
// v_mfma_f32_16x16x32_f16, so one instruction makes two of the three
// products:
//   N = 16: A = [R hi | R lo] against [T hi; T hi] and (DCT) [T lo; 0];
//   N = 8:  two nodes fill the 16 rows, both families the 16 columns, and
//           A = [R hi | R lo | R hi | 0] against [T hi; T hi; T lo; 0] makes
//           all three products at once.
// N = 16 carries the correlations from step to step as kernels_sep.hip does,
// until one of the wave's running nodes wants them anew (then all take them);
// with four nodes to a wave N = 8 would want them at most steps.  Largest
// error over ||r|| (as measured there): N = 16 5.3e-7, FP32 products of every
// step 2.2e-6; N = 8 3.5e-7.  Selection as there, too: every atom whose |c| is
// within 2^-13 ||r'|| of the largest is re-scored in FP64 (the bound holds with
// room: 48 FP32 additions at most per product instead of 192, and 5 2^-22 for
// the split of either); where they are many see kSubMany and kList.
//
// What bounds it: the instructions of a step (about 400 for the two nodes of
// a wave), then the longest pursuits.  On three 2048 x 2048 planes N = 16
// (157 690 node-steps) takes 86 us and N = 8 (170 692) 74 us; with the N = 16
// correlations made anew at every step, matrix-core results copied out of the
// accumulator registers and the constant atom's sums beside the others' 124
// and 88 us, with the unfactored BF16 product (8 or 4 times the operations)
// in workgroups of 16 slots, which met three times a step, 254 and 115 us.
// FP32 form, 1536 x 1024 x 3: N = 16 63 us (FP32 products at every step 97 us,
// step by step 1 870 us).
//
// N = 8 of the FP32 form (k_mp_fused) keeps the residual and its coefficients
// in FP64: the FP16 split only proposes the atoms, and a candidate's
// coefficient is the plain sum over the 64 pixels, one after the other, as if
// every atom had its own (c_a = <r, phi_a>, dense).  That chain of 64 FP64
// fused multiply-adds is a third of the step; its operands want registers, so
// two waves per SIMD measured best (70 us for the 476 nodes of a 512 x 512
// plane, 83 us for 4 544; four per SIMD 89 and 92 us).  The dense FP64 product
// with all atoms from LDS, a node per wave, took 78 and 215 us.
//
// The order of operations of the FP64 re-score, update and norms is fixed by
// the patches (SubGeo): BF16 form a slot of 32 (N = 16) or 16 lanes with rows
// of four pixels per lane; FP32 form k_select's and k_gather's, so that it
// equals the step-by-step form bit for bit; its N = 8 the sums over lane =
// pixel of the dense form.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

typedef _Float16 sb_h8 __attribute__((ext_vector_type(8)));
typedef float sb_f32x4 __attribute__((ext_vector_type(4)));

// The three forms: FP32 (N = 16), BF16 (N = 8 and 16), and the FP32 form's
// exact one (N = 8), whose residual stays FP64.
enum { SUB_F32, SUB_BF16, SUB_F64 };

template <int N_, int FAMS_, int FORM_>
struct SubGeo {
  static constexpr int N = N_, K = N * N, FAMS = FAMS_;
  static constexpr bool EXACT = FORM_ == SUB_F64;
  static constexpr bool BF = FORM_ != SUB_F32;            // the BF16 form's patches
  static constexpr int NFAM = FAMS == 3 ? 2 : 1;
  static constexpr int SN = BF ? (N == 16 ? 2 : 4) : 1;   // nodes per wave
  static constexpr int LPS = 64 / SN;                     // lanes per slot
  static constexpr int PC = BF ? 4 : 2;                   // patch: columns,
  static constexpr int PR = K / LPS / PC;                 // rows of a lane
  static constexpr int XQ = N / PC;                       // patches per row of patches
  // values per lane and node: N = 16 four per family; N = 8 four (rows and
  // columns of one family meet in half of the lanes)
  static constexpr int VPL = N == 16 ? 4 * NFAM : 4;
  // N = 16: correlations carried from step to step (N = 8: one of the four
  // nodes of a wave would want them anew at most steps)
  static constexpr bool CARRY = N == 16;
  // N = 8: several candidates of a node take a lane of its slot each
  static constexpr bool WIDE = N == 8;
  // operand row in LDS (value half, remainder half, padding against bank
  // conflicts), and bytes per node
  static constexpr int ROWB = N == 16 ? 80 : 48;
  static constexpr int NODEB = N * ROWB;
  static constexpr float TS = 128.f;                      // see SepGeo::TS
  static_assert((N == 16 && !EXACT) || (N == 8 && BF), "block sizes");
  static_assert(PR * PC * LPS == K && PR >= 1 && VPL <= 8, "patches");
};

__device__ inline uint32_t sb_split_hi(float a, float b) {
  const auto p = __builtin_amdgcn_cvt_pkrtz(a, b);
  uint32_t h;
  __builtin_memcpy(&h, &p, 4);
  return h;
}
// packed FP16 remainders of a pair (see sp_split2, also for the wait states)
__device__ inline uint32_t sb_split_lo(float a, float b, uint32_t h) {
  uint32_t l;
  __asm__("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(l) : "v"(h), "v"(a));
  __asm__("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]\n\ts_nop 1" : "+v"(l) : "v"(h), "v"(b));
  return l;
}

// Table operands: t1 the B operands of the first product, t2 the A operands of
// the second; index 0 the products with [T hi; T hi] (N = 8: all three), 1 the
// DCT's remainders.
template <class G>
struct SubOps {
  sb_h8 t1[G::N == 8 ? 1 : G::NFAM], t1l[1], t2[G::N == 8 ? 2 : G::NFAM], t2l[G::N == 8 ? 2 : 1];
  float sc[4];                                            // N = 16: Haar magnitudes of rows 4 g + r and the lane's column
};

template <class G>
__device__ constexpr bool sub_haar(int f) { return G::FAMS == AQMP_HAAR || (G::FAMS == 3 && f == 1); }

// tabs: the FP64 tables of the dictionary's families, [f][row][col].
template <class G>
__device__ inline void sub_load_ops(SubOps<G>& T, const double* tabs) {
  constexpr int N = G::N, K = G::K;
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  // operand value: scaled DCT entry, or Haar entry (its sign for N = 16)
  auto hi_lo = [](float v, _Float16& h, _Float16& l) {
    h = (_Float16)v;
    l = (_Float16)(v - (float)h);
  };
  if constexpr (N == 16) {
#pragma unroll
    for (int f = 0; f < G::NFAM; ++f) {
      const bool hr = sub_haar<G>(f);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // first product: k = 8 g + j is pixel x = k % 16 (value, then remainder of R)
        const double a = tabs[f * K + m * N + ((8 * g + j) & 15)];
        // second: k-slot (g, j) is row y = 4 g + j % 4 (value, then remainder of D1)
        const double b = tabs[f * K + m * N + 4 * g + (j & 3)];
        if (hr) {
          T.t1[f][j] = (_Float16)(a > 0.0 ? 1.f : (a < 0.0 ? -1.f : 0.f));
          T.t2[f][j] = (_Float16)(b > 0.0 ? 1.f : (b < 0.0 ? -1.f : 0.f));
        } else {
          _Float16 h, l;
          hi_lo((float)a * G::TS, h, l);
          T.t1[f][j] = h;
          T.t1l[0][j] = g < 2 ? l : (_Float16)0.f;
          hi_lo((float)b * G::TS, h, l);
          T.t2[f][j] = h;
          T.t2l[0][j] = j < 4 ? l : (_Float16)0.f;
        }
      }
      if (hr) {
        auto mag = [&](int row) -> float {
          int at = 0;
          if (row > 0) {
            const int top = 1 << (31 - __builtin_clz((unsigned)row));
            at = (row - top) * (N / top);
          }
          return (float)tabs[f * K + row * N + at];
        };
        const float mq = mag(m) * (G::TS * G::TS);
#pragma unroll
        for (int r = 0; r < 4; ++r) T.sc[r] = mag(4 * g + r) * mq;
      }
    }
  } else {
    // N = 8: column n = 8 f + q of the first product, row 8 f + p of the
    // second; all entries scaled values (no sign form).  k-slots of the
    // first: g = 0 (R hi) T hi, g = 1 (R lo) T hi, g = 2 (R hi) T lo, g = 3 zero;
    // of the second, for the node of rows g / 2 == u: (g, j) is row
    // y = 4 (g % 2) + j % 4 of D1's values, then remainders.
    const int fc = m >> 3, c = m & 7;
    const bool ok = fc < G::NFAM;
    const double* tf = tabs + (ok ? fc : 0) * K + c * N;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      _Float16 h, l;
      hi_lo(ok ? (float)tf[j] * G::TS : 0.f, h, l);
      T.t1[0][j] = g < 2 ? h : (g == 2 ? l : (_Float16)0.f);
      hi_lo(ok ? (float)tf[4 * (g & 1) + (j & 3)] * G::TS : 0.f, h, l);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        T.t2[u][j] = (g >> 1) == u ? h : (_Float16)0.f;
        T.t2l[u][j] = (g >> 1) == u && j < 4 ? l : (_Float16)0.f;
      }
    }
  }
}

// Correlations of the wave's nodes with all atoms, scaled by TS^2 and the
// node's row scale: V[n][v], atom_of(lane, v).
template <class G>
__device__ inline void sub_correlate(const char* sR, const SubOps<G>& T, float (&V)[G::SN][G::VPL]) {
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const sb_f32x4 z4{0.f, 0.f, 0.f, 0.f};
  if constexpr (G::N == 16) {
    sb_f32x4 D[G::SN][G::NFAM];
#pragma unroll
    for (int n = 0; n < G::SN; ++n) {
      const sb_h8 a = *(const sb_h8*)(sR + n * G::NODEB + m * G::ROWB + 16 * g);
#pragma unroll
      for (int f = 0; f < G::NFAM; ++f) {
        D[n][f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, T.t1[f], z4, 0, 0, 0);
        if (!sub_haar<G>(f)) D[n][f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, T.t1l[0], D[n][f], 0, 0, 0);
      }
    }
#pragma unroll
    for (int n = 0; n < G::SN; ++n)
#pragma unroll
      for (int f = 0; f < G::NFAM; ++f) {
        const sb_f32x4 d = D[n][f];
        uint32_t w[4];
        w[0] = sb_split_hi(d[0], d[1]);
        w[1] = sb_split_hi(d[2], d[3]);
        w[2] = sb_split_lo(d[0], d[1], w[0]);
        w[3] = sb_split_lo(d[2], d[3], w[1]);
        sb_h8 b;
        __builtin_memcpy(&b, w, 16);
        sb_f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_f16(T.t2[f], b, z4, 0, 0, 0);
        if (!sub_haar<G>(f)) c = __builtin_amdgcn_mfma_f32_16x16x32_f16(T.t2l[0], b, c, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) V[n][4 * f + r] = sub_haar<G>(f) ? c[r] * T.sc[r] : c[r];
      }
  } else {
    sb_f32x4 D[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {   // nodes 2 u and 2 u + 1: 16 rows
      const sb_h8 a = *(const sb_h8*)(sR + 2 * u * G::NODEB + m * G::ROWB + (g == 1 ? 16 : 0));
      D[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, T.t1[0], z4, 0, 0, 0);
    }
    const bool on = (g >> 1) == (m >> 3);   // rows and columns of one family
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const sb_f32x4 d = D[u];
      uint32_t w[4];
      w[0] = sb_split_hi(d[0], d[1]);
      w[1] = sb_split_hi(d[2], d[3]);
      w[2] = sb_split_lo(d[0], d[1], w[0]);
      w[3] = sb_split_lo(d[2], d[3], w[1]);
      sb_h8 b;
      __builtin_memcpy(&b, w, 16);
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        sb_f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_f16(T.t2[v], b, z4, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(T.t2l[v], b, c, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) V[2 * u + v][r] = on ? c[r] : 0.f;
      }
    }
  }
}

// Atom of value v in lane l (see sub_correlate).
template <class G>
__device__ inline int sub_atom(int l, int v) {
  const int m = l & 15, g = l >> 4;
  if constexpr (G::N == 16) return (v >> 2) * G::K + m * 16 + 4 * g + (v & 3);
  else return (m >> 3) * G::K + (m & 7) * 8 + 4 * (g & 1) + v;
}

// Sum over the lanes of a slot, a butterfly (every lane gets the same bits).
template <class G>
__device__ inline double sub_slot_sum(double v) {
  if constexpr (G::LPS == 64) {
    return wave_sum_f64(v);
  } else {
    if constexpr (G::EXACT) {            // pixels in the order of their bits
      v += row_perm_f64<0xB1>(v);
      v += row_perm_f64<0x4E>(v);
      v += row_perm_f64<0x141>(v);
      v += row_perm_f64<0x128>(v);
      return v;
    }
    if constexpr (G::LPS == 32) v = lane_pair_sum_f64<16>(v);
    v += row_perm_f64<0x128>(v);   // row_ror:8
    v += row_perm_f64<0x141>(v);   // row_half_mirror
    v += row_perm_f64<0x4E>(v);    // quad_perm [2,3,0,1]
    v += row_perm_f64<0xB1>(v);    // quad_perm [1,0,3,2]
    return v;
  }
}

// The atom of the largest correlation of a node of N = 16, in FP64 from its FP32
// pixels (rows of ROWB bytes), the lowest within w: see sep_exact.
template <class G>
__device__ inline int sub_exact(const char* px, const double* tab, double w) {
  constexpr int N = G::N, K = G::K;
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  LaneBest best;
#pragma unroll 1
  for (int f = 0; f < G::NFAM; ++f) {
    const double* row = tab + (f * N + m) * N + g;
    d4 D = d4{0.0, 0.0, 0.0, 0.0}, c = D;
#pragma unroll 1
    for (int x = 0; x < N; x += 4) D = mfma64((double)((const float*)(px + m * G::ROWB))[x + g], row[x], D);
#pragma unroll
    for (int y = 0; y < N; y += 4) {
      c = mfma64(row[y], D[y / 4], c);
      __asm__ volatile("" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]) : : "memory");
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int at = f * K + m * N + g + 4 * r;
      best.take(f == 1 && at == K ? 0.0 : c[r], at, w);   // (the second constant atom)
    }
  }
  best.over_wave(w);
  return best.atom;
}

// N = 16: more lanes than this with a candidate of one node, and its
// correlations are made in FP64 (256 x 256 checkered, Haar alone, 16 steps:
// 66 us, 348 with all candidates re-scored in turn).
constexpr int kSubMany = 8;
// N = 8 re-scores them all.  The BF16 form takes up to this many in turn, its
// lanes summing one together; more, and in the FP32 form any second one, at once,
// a lane each with the same sums.  The same plane: 74 us BF16 and 75 FP32, 98
// and 127 with all in turn; binary text, two families, 55 and 72 (56 and 69: two
// candidates are the FP32 form's best case in turn).
constexpr int kList = 5;

template <class G>
__device__ inline void pursuit_sub(const JobDev* __restrict__ jobs, const LevelDev& lv,
                                   const int32_t* __restrict__ count_ptr, int32_t* __restrict__ queue,
                                   const double* __restrict__ tab, const double* __restrict__ xg) {
  constexpr int N = G::N, K = G::K, SN = G::SN, LPS = G::LPS, PR = G::PR, PC = G::PC, VPL = G::VPL;
  constexpr bool BF = G::BF, EXACT = G::EXACT;
  constexpr int lg = N == 16 ? 4 : 3;
  // rows of the families' tables, then a row of ones and one of 1/N: the
  // constant atom's factors
  constexpr int ONES = G::NFAM * N;
  __shared__ __attribute__((aligned(16))) double sTab[ONES + 2][N];
  __shared__ __attribute__((aligned(16))) char sRows[4][SN * G::NODEB];
  // CARRY: FP32 <T_f[p], T_f'[p']> of the step's family f and each f'
  __shared__ __attribute__((aligned(16))) float sX[G::CARRY ? G::NFAM : 1][G::NFAM][G::CARRY ? N : 1][G::CARRY ? N : 1];
  // WIDE: the residuals in FP64 (EXACT at every step, else for steps with
  // several candidates), every slot's on banks of its own, and its candidates
  constexpr bool WIDE = G::WIDE;
  constexpr int RP = K + 2;
  __shared__ __attribute__((aligned(16))) double sPix[WIDE ? 4 : 1][WIDE ? SN * RP : 2];
  __shared__ uint8_t sCand[WIDE ? 4 : 1][WIDE ? SN : 1][WIDE ? 2 * K : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* sR = sRows[wv];
  for (int i = tid; i < G::NFAM * K; i += 256) (&sTab[0][0])[i] = tab[i];
  if (tid < 2 * N) sTab[ONES + tid / N][tid % N] = tid < N ? 1.0 : 1.0 / N;
  if constexpr (G::CARRY) {
    for (int i = tid; i < G::NFAM * G::NFAM * K; i += 256) {
      const int f = i / (G::NFAM * K), f2 = i / K % G::NFAM, a = i / N % N, b = i % N;
      float v = a == b ? 1.f : 0.f;
      if (f != f2) v = (float)(f == 0 ? xg[a * N + b] : xg[b * N + a]);
      sX[f][f2][a][b] = v;
    }
  }
  for (int i = lane; i < SN * G::NODEB / 16; i += 64) ((uint4*)sR)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  SubOps<G> T;
  sub_load_ops<G>(T, &sTab[0][0]);
  const int count = *count_ptr;
  const int slot = lane / LPS, li = lane % LPS;
  const int py = (li / G::XQ) * PR, px = (li % G::XQ) * PC;
  char* sRow = sR + slot * G::NODEB;
  // The first nodes are dealt out in order, the others by the queues.
  const int q0 = (int)gridDim.x * 4 * SN, qk = (int)blockIdx.x % kQueues;
  int node = ((int)blockIdx.x * 4 + wv) * SN + slot;
  int ahead = 0;                       // the slot's next node (its first lane)
  bool dry = node >= count, run = false, load = !dry;
  int t = 0, kmax = 0, rec_i = 0;
  double rec_c = 0.0, e = 0.0, eps2 = 0.0;
  double sc = 1.0;
  float win = 0.f;
  // the carried correlations hold while e is in [elim, emax) and t < tlim
  bool fresh = false;
  double elim = 0.0, emax = 0.0;
  int tlim = 0;
  float V[SN][VPL];
#pragma unroll
  for (int n = 0; n < SN; ++n)
#pragma unroll
    for (int v = 0; v < VPL; ++v) V[n][v] = 0.f;
  double rd[PR][PC];
#pragma unroll
  for (int i = 0; i < PR; ++i)
#pragma unroll
    for (int j = 0; j < PC; ++j) rd[i][j] = 0.0;

  // see k_pursuit_sep; FP64, so that no norm of FP32 pixels is out of its range
  auto scale_of = [](double en) -> double {
    const int ex = (int)((unsigned long long)__double_as_longlong(en) >> 52) - 1023;
    const int sh = (ex >> 1) - 7;
    return __longlong_as_double((long long)(1023 - sh) << 52);
  };
  // EXACT: ||r||^2 beyond what the ranking's scale can take (an FP64 plane's
  // extremes): every atom is a candidate
  auto beyond = [](double en) { return EXACT && !(en >= 0x1p-900 && en < 0x1p900); };
  auto still = [&](double en) {              // nothing to select: a zero residual, or undefined pixels
    if constexpr (!EXACT) return !(en > 0.0 && en < __builtin_inf());
    bool any = false;
#pragma unroll
    for (int i = 0; i < PR; ++i)
#pragma unroll
      for (int j = 0; j < PC; ++j) any = any || rd[i][j] != 0.0;
    const unsigned long long lanes = __ballot(any) >> (lane & ~(LPS - 1));
    return !(en < __builtin_inf()) || (lanes & ((1ull << (LPS % 64)) - 1ull)) == 0ull;
  };
  // Some pixel of the slot's node, finite in FP64, is not in FP32.
  auto past_f32 = [&]() {
    bool any = false;
#pragma unroll
    for (int i = 0; i < PR; ++i)
#pragma unroll
      for (int j = 0; j < PC; ++j) any = any || !(fabs(rd[i][j]) < __builtin_inf());
    const unsigned long long lanes = __ballot(any) >> (lane & ~(LPS - 1));
    return (lanes & ((1ull << (LPS % 64)) - 1ull)) != 0ull;
  };
  // N = 8: two nodes meet in the second product, each masked from the other by
  // zeros of the table, which hide finite values only.  So no row of a slot is
  // ever infinite or undefined: such a node selects nothing, and what is put is
  // scaled by its norm.
  auto put_rows = [&]() {
#pragma unroll
    for (int i = 0; i < PR; ++i) {
      char* row = sRow + (py + i) * G::ROWB;
      float v[PC];
#pragma unroll
      for (int j = 0; j < PC; ++j) v[j] = (float)(rd[i][j] * sc);
      const uint32_t h0 = sb_split_hi(v[0], v[1]);
      if constexpr (PC == 4) {
        const uint32_t h1 = sb_split_hi(v[2], v[3]);
        *(uint2*)(row + 2 * px) = make_uint2(h0, h1);
        *(uint2*)(row + 2 * N + 2 * px) = make_uint2(sb_split_lo(v[0], v[1], h0), sb_split_lo(v[2], v[3], h1));
      } else {
        *(uint32_t*)(row + 2 * px) = h0;
        *(uint32_t*)(row + 2 * N + 2 * px) = sb_split_lo(v[0], v[1], h0);
      }
    }
  };

  // EXACT: the first two levels of the norm's butterfly over the pixels
  auto quad = [](const double (&v)[PC]) -> double {
    return fma(v[0], v[0], v[1] * v[1]) + fma(v[PC - 2], v[PC - 2], v[PC - 1] * v[PC - 1]);
  };

  for (;;) {
    // ---- slots without a node take their next one ----
    if (__ballot(load) != 0ull) {
      if (load) {
        const int jidx = lv.job[node];
        const int bx = lv.x0[node], by = lv.y0[node];
        const JobDev jl = jobs[jidx];
        eps2 = jobs[jidx].eps2[lg];
        kmax = jobs[jidx].k[lg];
        if constexpr (BF) {
          double pv[PR][PC];
#pragma unroll
          for (int i = 0; i < PR; ++i) job_pixels<PC>(jl, by + py + i, bx + px, pv[i]);
          double ep = 0.0;
#pragma unroll
          for (int i = 0; i < PR; ++i) {
            double ei = 0.0;
#pragma unroll
            for (int j = 0; j < PC; ++j) {
              rd[i][j] = EXACT ? pv[i][j] : (double)(float)pv[i][j];
              ei = fma(pv[i][j], pv[i][j], ei);
            }
            ep += EXACT ? quad(pv[i]) : ei;
          }
          e = sub_slot_sum<G>(ep);
        } else {
          // k_gather's layout: one pixel per thread of four waves
          double gv[4], pv[PR][PC];
#pragma unroll
          for (int w = 0; w < 4; ++w) gv[w] = job_pixel(jl, by + 4 * w + (lane >> 4), bx + (lane & 15));
#pragma unroll
          for (int i = 0; i < PR; ++i) job_pixels<PC>(jl, by + py + i, bx + px, pv[i]);
#pragma unroll
          for (int i = 0; i < PR; ++i)
#pragma unroll
            for (int j = 0; j < PC; ++j) rd[i][j] = (double)(float)pv[i][j];
          double s[4];
#pragma unroll
          for (int w = 0; w < 4; ++w) s[w] = wave_sum_f64(gv[w] * gv[w]);
          e = (s[0] + s[1]) + (s[2] + s[3]);
        }
        t = 0;
        uint8_t st = ST_RUN;
        if (e < eps2)
          st = ST_ACC;
        else if (kmax <= 0)
          st = ST_SPARSE;
        else if (still(e))
          st = ST_ZERO;
        if constexpr (N == 8 && !EXACT) {
          if (past_f32() && st == ST_RUN) st = ST_ZERO;
        }
        run = st == ST_RUN;
        fresh = true;
        if (!run && li == 0) {
          lv.e[node] = e;
          lv.t[node] = 0;
          lv.st[node] = st;
        }
      }
    }
    const unsigned long long runs = __ballot(run);
    if (runs != 0ull) {
      // ---- correlations, from the residual or carried ----
      if (!G::CARRY || __ballot(run && fresh) != 0ull) {
        if (run) {
          sc = beyond(e) ? 0.0 : scale_of(e);
          put_rows();
          if constexpr (EXACT) {
#pragma unroll
            for (int j = 0; j < PC; j += 2)
              *(double2*)&sPix[wv][slot * RP + N * py + px + j] = make_double2(rd[0][j], rd[0][j + 1]);
          }
          win = __builtin_amdgcn_sqrtf((float)(e * sc * sc)) * (1.0001f * 0x1p-13f * G::TS * G::TS);
          elim = fmax(eps2, 0.25 * e);
          emax = 4.0 * e;
          tlim = t + 64 < kmax ? t + 64 : kmax;
        }
        wave_sync();
        sub_correlate<G>(sR, T, V);
        wave_sync();   // the rows are read before any slot writes new ones
      }
      if constexpr (G::NFAM == 2) {
        // the second family's constant atom equals the first's, which wins the tie
        const bool dc1 = lane == (N == 16 ? 0 : 40);
        constexpr int v1 = N == 16 ? 4 : 0;
#pragma unroll
        for (int n = 0; n < SN; ++n) V[n][v1] = dc1 ? 0.f : V[n][v1];
      }
      // ---- per node the atoms within the window of its largest ----
      const unsigned long long far = EXACT ? __ballot(run && beyond(e)) : 0ull;
      unsigned long long lanes[SN];
      uint32_t mask[SN], bits[SN];
      bool more = false;
      uint32_t many = 0u;              // nodes with candidates in more than kSubMany lanes
      int cand = 0;
#pragma unroll
      for (int n = 0; n < SN; ++n) {
        float m0 = 0.f;
#pragma unroll
        for (int v = 0; v < VPL; v += 2) m0 = fmaxf(fmaxf(fabsf(V[n][v]), fabsf(V[n][v + 1])), m0);
        const float mx = wave_max_f32(m0);
        const float wn = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(win), n * LPS));
        const float thr = mx - wn;
        uint32_t mk = 0u;
#pragma unroll
        for (int v = 0; v < VPL; ++v) mk = __builtin_amdgcn_alignbit(mk, __float_as_uint(thr - fabsf(V[n][v])), 31);
        // a slot at rest, or infinite or undefined sums: nothing to compare
        const bool on = ((runs >> (n * LPS)) & 1ull) != 0ull;
        const bool alive = on && mx > 0.f && mx < __builtin_inff();
        mask[n] = alive ? mk : 0u;
        if constexpr (EXACT) {
          const int fm = (lane & 15) >> 3;
          if ((far >> (n * LPS)) & 1ull) mask[n] = on && (lane >> 5) == fm && fm < G::NFAM ? (1u << VPL) - 1u : 0u;
        }
        lanes[n] = __ballot(mask[n] != 0u);
        if constexpr (!WIDE) {
          if (__popcll(lanes[n]) > kSubMany) {
            many |= 1u << n;
            lanes[n] = 0ull;
          }
        }
        // the first candidate; whether there are others
        const int l = lanes[n] ? __builtin_ctzll(lanes[n]) : 0;
        bits[n] = (uint32_t)__builtin_amdgcn_readlane((int)mask[n], l);
        int at = -1;
        if (lanes[n]) {
          at = sub_atom<G>(l, VPL - 1 - __builtin_ctz(bits[n]));
          bits[n] &= bits[n] - 1u;
          if (bits[n] == 0u) lanes[n] &= lanes[n] - 1ull;
          more = more || lanes[n] != 0ull;
        }
        cand = slot == n ? at : cand;
      }
      if (!WIDE && many) {
        do {
          const int n = __builtin_ctz(many);
          many &= many - 1u;
          if (slot == n) {
#pragma unroll
            for (int i = 0; i < PR; ++i)
#pragma unroll
              for (int j = 0; j < PC; ++j) ((float*)(sRow + (py + i) * G::ROWB))[px + j] = (float)rd[i][j];
          }
          wave_sync();
          const int at = sub_exact<G>(sR + n * G::NODEB, &sTab[0][0], 0x1p-42 * __builtin_sqrt(lane_f64(e, n * LPS)));
          wave_sync();
          cand = slot == n ? at : cand;
        } while (many);
        // the correlations anew: kept over the products they were 23 registers
        // too many (BF16, both families)
        if (run) put_rows();
        wave_sync();
        sub_correlate<G>(sR, T, V);
        wave_sync();
      }
      // ---- FP64 re-score of the slot's candidate ----
      double tq[PC], tp[PR];
      auto rows = [&](int a) {
        const int f = a / K, q = (a % K) / N, p = a % N;
        const bool dc = (a % K) == 0;
        const double* tr = &sTab[dc ? ONES : f * N + q][px];
        const double* pr = &sTab[dc ? ONES + 1 : f * N + p][py];
#pragma unroll
        for (int j = 0; j < PC; j += 2) {
          const double2 v = *(const double2*)(tr + j);
          tq[j] = v.x;
          tq[j + 1] = v.y;
        }
#pragma unroll
        for (int i = 0; i < PR; ++i) tp[i] = pr[i];
      };
      // WIDE: the correlation of the slot's residual with any lane's atom a, EXACT
      // as the plain sum over the pixels, one after the other,
      auto plain = [&](int a) -> double {
        const int f = a / K, q = (a % K) / N, p = a % N;
        const bool dc = (a % K) == 0;
        const double* tr = sTab[dc ? ONES : f * N + q];
        const double* pr = sTab[dc ? ONES + 1 : f * N + p];
        double tx[N], c = 0.0;
#pragma unroll
        for (int x = 0; x < N; x += 2) {
          const double2 v = *(const double2*)(tr + x);
          tx[x] = v.x;
          tx[x + 1] = v.y;
        }
#pragma unroll
        for (int y = 0; y < N; ++y) {
          const double ty = pr[y];
#pragma unroll
          for (int x = 0; x < N; x += 2) {
            const double2 v = *(const double2*)&sPix[wv][slot * RP + N * y + x];
            c = fma(v.x, ty * tx[x], c);
            c = fma(v.y, ty * tx[x + 1], c);
          }
        }
        return c;
      };
      // else as the sums that the slot's lanes make together (see rescore and
      // sub_slot_sum): lane l holds row l / 2, columns 4 (l % 2) ..; its part is
      // added to those of l ^ 8, l ^ 7, l ^ 2 and l ^ 1 in turn.  (A few loads at
      // a time: with all at once 60 registers too many.)
      auto of_slot = [&](int a) __attribute__((always_inline)) -> double {
        const int f = a / K, q = (a % K) / N, p = a % N;
        const bool dc = (a % K) == 0;
        const double* tr = sTab[dc ? ONES : f * N + q];
        const double* pr = sTab[dc ? ONES + 1 : f * N + p];
        const double* pix = &sPix[wv][slot * RP];
        double h[8];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const double2 t0 = *(const double2*)(tr + 4 * s), t1 = *(const double2*)(tr + 4 * s + 2);
          auto part = [&](int y) __attribute__((always_inline)) -> double {
            const double2 u = *(const double2*)(pix + 8 * y + 4 * s), v = *(const double2*)(pix + 8 * y + 4 * s + 2);
            return fma(pr[y], fma(u.x, t0.x, u.y * t0.y) + fma(v.x, t1.x, v.y * t1.y), 0.0);
          };
#pragma unroll
          for (int y = 0; y < 4; ++y) {
            h[2 * y + s] = part(y) + part(y + 4);
            __asm__ volatile("" : "+v"(h[2 * y + s]));   // made here, not where the sum is used
          }
        }
        return ((h[0] + h[7]) + (h[2] + h[5])) + ((h[1] + h[6]) + (h[3] + h[4]));
      };
      auto rescore = [&](int a) -> double {   // a >= 0
        rows(a);
        if constexpr (EXACT) return plain(a);
        double part = 0.0;
#pragma unroll
        for (int i = 0; i < PR; ++i) {
          double sy;
          if constexpr (BF) {
            sy = fma(rd[i][0], tq[0], rd[i][1] * tq[1]) + fma(rd[i][2], tq[2], rd[i][3] * tq[3]);
          } else {
            sy = 0.0;
#pragma unroll
            for (int j = 0; j < PC; ++j) sy = fma(rd[i][j], tq[j], sy);
          }
          part = fma(tp[i], sy, part);   // (a product would be fused into the slot sum)
        }
        return sub_slot_sum<G>(part);
      };
      int atom = cand;
      double coef = rescore(cand < 0 ? 0 : cand);
      double mag = cand < 0 ? 0.0 : fabs(coef);
      bool lists = EXACT && more;      // (taken in turn beside it, the step itself was slower)
      if (WIDE && !EXACT && more) {
#pragma unroll
        for (int n = 0; n < SN; ++n) {
          if (!lanes[n]) continue;
          int cnt = 0;
#pragma unroll
          for (int v = 0; v < VPL; ++v) cnt += __popcll(__ballot(((mask[n] >> v) & 1u) != 0u));
          lists = lists || cnt > kList;
        }
      }
      if (lists) {
        // All atoms of a node, sixteen at a time, a lane of the slot each, lowest
        // index on ties.
        int total = 0;
#pragma unroll
        for (int n = 0; n < SN; ++n) {
          if (!EXACT && !lanes[n]) continue;   // one candidate or none: done
          int cnt = 0;
#pragma unroll
          for (int v = 0; v < VPL; ++v) {
            const bool b = ((mask[n] >> (VPL - 1 - v)) & 1u) != 0u;
            const unsigned long long m = __ballot(b);
            if (b) sCand[wv][n][cnt + __popcll(m & ((1ull << lane) - 1ull))] = (uint8_t)sub_atom<G>(lane, v);
            cnt += __popcll(m);
          }
          total = slot == n ? cnt : total;
        }
        if constexpr (!EXACT) {
#pragma unroll
          for (int j = 0; j < PC; j += 2)
            *(double2*)&sPix[wv][slot * RP + N * py + px + j] = make_double2(rd[0][j], rd[0][j + 1]);
        }
        wave_sync();
        double bm = 0.0, bc = 0.0;
        int ba = 0x7fffffff;
        for (int i = li; __ballot(i < total) != 0ull; i += LPS) {
          if constexpr (!EXACT) __asm__ volatile("" ::: "memory");   // no pixels kept in registers from pass to pass
          const int a = i < total ? (int)sCand[wv][slot][i] : 0;
          const double c0 = EXACT ? plain(a) : of_slot(a), m0 = fabs(c0);
          if (i < total && (m0 > bm || (m0 == bm && a < ba))) {
            bm = m0;
            bc = c0;
            ba = a;
          }
        }
        const unsigned long long mb = (unsigned long long)__double_as_longlong(bm), m = row_max_u64(mb);
        const int at = row_min_i32(mb == m ? ba : 0x7fffffff);
        const double c1 = sub_slot_sum<G>(mb == m && ba == at ? bc : 0.0);
        if (EXACT || total > 0) {
          mag = __longlong_as_double((long long)m);
          coef = c1;
          atom = at == 0x7fffffff ? -1 : at;
        }
        rows(atom < 0 ? 0 : atom);
        wave_sync();   // the lists are read before a later step writes them
      } else if (!EXACT && more) {
        // the other atoms of the windows, lowest index on ties
        while (more) {
          more = false;
          int at = -1;
#pragma unroll
          for (int n = 0; n < SN; ++n) {
            int an = -1;
            if (lanes[n]) {
              const int l = __builtin_ctzll(lanes[n]);
              if (bits[n] == 0u) bits[n] = (uint32_t)__builtin_amdgcn_readlane((int)mask[n], l);
              an = sub_atom<G>(l, VPL - 1 - __builtin_ctz(bits[n]));
              bits[n] &= bits[n] - 1u;
              if (bits[n] == 0u) lanes[n] &= lanes[n] - 1ull;
              more = more || lanes[n] != 0ull;
            }
            at = slot == n ? an : at;
          }
          const double c0 = rescore(at < 0 ? 0 : at), m0 = fabs(c0);
          const bool take = at >= 0 && (m0 > mag || (m0 == mag && at < atom));
          mag = take ? m0 : mag;
          coef = take ? c0 : coef;
          atom = take ? at : atom;
        }
        rows(atom < 0 ? 0 : atom);
      }
      // ---- rank-1 update, norm, record, stop test ----
      uint8_t st = ST_RUN;
      const bool zero = !(mag > 0.0);
      double en = 0.0;
#pragma unroll
      for (int i = 0; i < PR; ++i) {
        double ei = 0.0;
#pragma unroll
        for (int j = 0; j < PC; ++j) {
          const double rx = fma(-coef, tp[i] * tq[j], rd[i][j]);
          const double rn = EXACT ? rx : (double)(float)rx;
          rd[i][j] = rn;               // a slot with nothing to select ends here
          ei = fma(rn, rn, ei);
        }
        en += EXACT ? quad(rd[i]) : ei;
      }
      if constexpr (G::CARRY) {
        // see k_pursuit_sep: c X[p][p'] X[q][q'] less, the own family's X the identity
        const float cs = (float)(coef * (sc * (double)(G::TS * G::TS)));
#pragma unroll
        for (int n = 0; n < SN; ++n) {
          const int an = __builtin_amdgcn_readlane(atom < 0 ? 0 : atom, n * LPS);
          const float cn = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(cs), n * LPS));
          const int f = an / K, q = (an % K) / N, p = an % N;
#pragma unroll
          for (int f2 = 0; f2 < G::NFAM; ++f2) {
            const float gq = -(cn * sX[f][f2][q][lane & 15]);
            const sb_f32x4 gp = *(const sb_f32x4*)&sX[f][f2][p][4 * (lane >> 4)];
#pragma unroll
            for (int r = 0; r < 4; ++r) V[n][4 * f2 + r] = fmaf(gq, gp[r], V[n][4 * f2 + r]);
          }
        }
      }
      en = sub_slot_sum<G>(en);
      const bool none = still(en);
      if (run) {
        if (zero) {
          st = ST_ZERO;
        } else {
          e = en;
          if (li == (t & (LPS - 1))) {
            rec_i = atom;
            rec_c = coef;
          }
          ++t;
          if (e < eps2)
            st = ST_ACC;
          else if (t >= kmax)
            st = ST_SPARSE;
          else if (none)
            st = ST_ZERO;
          fresh = !(e >= elim && e < emax && t < tlim);
          const int base = (t - 1) & ~(LPS - 1);   // first step held in the registers
          if (st != ST_RUN || t - base == LPS) {
            if (li < t - base) {
              const size_t rs = (size_t)node * lv.kmax + base + li;
              lv.rec_idx[rs] = rec_i;
              lv.rec_coef[rs] = rec_c;
            }
          }
        }
        if (zero) {
          const int base = t & ~(LPS - 1);
          if (li < t - base) {
            const size_t rs = (size_t)node * lv.kmax + base + li;
            lv.rec_idx[rs] = rec_i;
            lv.rec_coef[rs] = rec_c;
          }
        }
        if (st != ST_RUN && li == 0) {
          lv.e[node] = e;
          lv.t[node] = t;
          lv.st[node] = st;
        }
        run = st == ST_RUN;
      }
    }
    // ---- the next node of the slots that ended ----
    load = false;
    if (__ballot(!run && !dry) != 0ull) {
      if (!run && !dry && li == 0) ahead = atomicAdd(queue + qk * kQueuePad, 1);   // (not before: see k_pursuit_sep)
      const int idx = q0 + __shfl(ahead, lane & ~(LPS - 1), 64) * kQueues + qk;
      if (!run && !dry) {
        node = idx;
        dry = idx >= count;
        load = !dry;
      }
    }
    if (__ballot(run || load) == 0ull) break;
  }
}

// (Four waves per SIMD, not any number: the matrix cores then write ordinary registers.)
template <int N, int FAMS>
__global__ __launch_bounds__(256, 4) void k_pursuit_bf16(const JobDev* __restrict__ jobs, LevelDev lv,
                                                      const int32_t* __restrict__ count_ptr,
                                                      int32_t* __restrict__ queue, const double* __restrict__ tab,
                                                      const double* __restrict__ xg) {
  pursuit_sub<SubGeo<N, FAMS, SUB_BF16>>(jobs, lv, count_ptr, queue, tab, xg);
}

template <int FAMS>
__global__ __launch_bounds__(256, 4) void k_pursuit16_f32(const JobDev* __restrict__ jobs, LevelDev lv,
                                                       const int32_t* __restrict__ count_ptr,
                                                       int32_t* __restrict__ queue, const double* __restrict__ tab,
                                                       const double* __restrict__ xg) {
  pursuit_sub<SubGeo<16, FAMS, SUB_F32>>(jobs, lv, count_ptr, queue, tab, xg);
}

// (Two waves per SIMD: see the head.)
template <int N, int FAMS>
__global__ __launch_bounds__(256, 2) void k_mp_fused(const JobDev* __restrict__ jobs, LevelDev lv,
                                                  const int32_t* __restrict__ count_ptr, int32_t* __restrict__ queue,
                                                  const double* __restrict__ tab, const double* __restrict__ xg) {
  pursuit_sub<SubGeo<N, FAMS, SUB_F64>>(jobs, lv, count_ptr, queue, tab, xg);
}

// As many workgroups as are resident at once, at most one per 4 SN nodes.
template <class Kern>
hipError_t launch_sub(Kern kern, int nodes_per_wg, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue,
                      int64_t cap, const double* tab, const double* xg, hipStream_t s) {
  int dev = 0, n_cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, 0) != hipSuccess || per_cu < 1) per_cu = 1;
  int64_t wgs = (cap + nodes_per_wg - 1) / nodes_per_wg;
  if (wgs > (int64_t)n_cus * per_cu) wgs = (int64_t)n_cus * per_cu;
  if (wgs < 1) wgs = 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), 0, s, jobs, lv, count, queue, tab, xg);
  return hipGetLastError();
}

template <int FAMS>
hipError_t launch_sub_f(int n, int precision, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue,
                        int64_t cap, const double* tab, const double* xg, hipStream_t s) {
  if (precision == AQMP_PREC_BF16) {
    if (n == 8) return launch_sub(k_pursuit_bf16<8, FAMS>, 4 * SubGeo<8, FAMS, SUB_BF16>::SN, jobs, lv, count, queue, cap, tab, xg, s);
    if (n == 16) return launch_sub(k_pursuit_bf16<16, FAMS>, 4 * SubGeo<16, FAMS, SUB_BF16>::SN, jobs, lv, count, queue, cap, tab, xg, s);
  } else if (n == 8) {
    return launch_sub(k_mp_fused<8, FAMS>, 4 * SubGeo<8, FAMS, SUB_F64>::SN, jobs, lv, count, queue, cap, tab, xg, s);
  } else if (n == 16) {
    return launch_sub(k_pursuit16_f32<FAMS>, 4, jobs, lv, count, queue, cap, tab, xg, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_pursuit_sub(int n, int precision, uint32_t families, const JobDev* jobs, LevelDev lv,
                              const int32_t* count, int32_t* queue, int64_t cap, const double* tab, const double* xg, hipStream_t s) {
  switch (families) {
    case AQMP_DCT: return launch_sub_f<AQMP_DCT>(n, precision, jobs, lv, count, queue, cap, tab, xg, s);
    case AQMP_HAAR: return launch_sub_f<AQMP_HAAR>(n, precision, jobs, lv, count, queue, cap, tab, xg, s);
    case AQMP_DCT | AQMP_HAAR: return launch_sub_f<AQMP_DCT | AQMP_HAAR>(n, precision, jobs, lv, count, queue, cap, tab, xg, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace aqmp
