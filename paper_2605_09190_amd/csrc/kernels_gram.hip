// kernels_gram.hip - Matching Pursuit through the Gram matrix (exact
// reformulation of Section 2.2, FP64 throughout), and Orthogonal Matching
// Pursuit in the same space.
//
// Every atom of D_N is an outer product of two rows of a 1D orthonormal table
// (Section 2.1), so
//   * the correlations of a block with all atoms of family f are the entries
//     of T_f Y T_f^T (two N x N products, O(N^3) per node instead of the
//     O(N^4) dense product), and
//   * after atom i is chosen with c_i = <r, phi_i>, the residual update
//     r <- r - c_i phi_i changes every correlation by the Gram column:
//     c_a <- c_a - c_i <phi_a, phi_i>, with
//     <phi_a, phi_i> = <T_fa[p_a], T_fi[p_i]> <T_fa[q_a], T_fi[q_i]>,
//     and the squared norm by e <- e - c_i^2 (phi_i has unit norm).
// The same-family part of that column is a Kronecker delta (each family is
// an orthonormal basis); the cross-family part is a product of two entries of
// the N x N table X[p][p'] = <T_0[p], T_1[p']>, built once with the
// dictionary with its row and column 0 exact (the constant rows are equal,
// every other row sums to zero).  So an MP step costs O(M) table lookups and
// FMAs, the residual itself is never formed, and the constant atoms (exactly
// 1/N) are handled exactly.
//
// k_gram_pursuit: a node's whole MP in one launch: the initial correlations as
// two FP64 matrix-core products per family (Z^T = Y^T T_f^T, then C^T = T_f
// Z^T), then the pursuit (selection with the lowest index on ties, records,
// stop test of eq. (2)) with the correlations held in registers.
// k_gram_init: gather, ||y||^2, the first stop test and the same products,
// written to a per-node buffer for the OMP kernel.  N / 16 waves per node,
// each owning one 16-wide strip of the row index p.
#include <type_traits>

#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

// LDS index of element (row, col) of an N x N FP64 tile.  The matrix-core
// operands are read as four rows of 16 consecutive doubles; for N >= 32 the
// odd rows swap their 16-column halves so that two such rows fall on
// different banks.
template <int N>
__device__ inline int sw(int row, int col) {
  if constexpr (N >= 32)
    return row * N + (col ^ ((row & 1) << 4));
  else
    return row * N + col;
}

template <int N, int NFAM>
struct InitGeo {
  static constexpr int K = N * N;
  static constexpr int M = NFAM * K;
  static constexpr int WPN = N / 16;        // waves per node
  static constexpr int GPW = 4 / WPN;       // nodes per workgroup
  static constexpr int TPN = 64 * WPN;      // threads per node
  static constexpr int T = N / 16;          // 16 x 16 output tiles along x (or p)
  static constexpr int KS = N / 4;          // k-steps of one product
};

// Wave wn of a node owns the 16-row strip s0 = 16 wn of the 1D tables.  It
// computes Z^T[x][p] for p in its strip (first product, all x) and C^T[q][p]
// for q in its strip (second product, all p).  Both products read the same
// table entries T_f[s0 + l % 16][4 ks + l / 16] (the B operand of the first,
// the A operand of the second), which the lane keeps in registers for the
// whole kernel; only Y and Z^T go through LDS.
template <int N, int NFAM>
__global__ __launch_bounds__(256) void k_gram_init(const JobDev* __restrict__ jobs, LevelDev lv,
                                                   const int32_t* __restrict__ count_ptr, int32_t lg,
                                                   const double* __restrict__ tab, double* __restrict__ cbuf) {
  using G = InitGeo<N, NFAM>;
  constexpr int K = G::K, M = G::M, WPN = G::WPN, GPW = G::GPW, TPN = G::TPN, T = G::T, KS = G::KS;
  __shared__ double sY[GPW][K];             // sY[g][sw(y, x)] = pixel (y, x)
  __shared__ double sZt[GPW][K];            // sZt[g][sw(x, p)] = (T_f Y)[p][x]
  __shared__ double sRed[GPW][WPN][2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = tid / TPN, tn = tid % TPN, wn = tn >> 6;
  const int s0 = 16 * wn;
  const int li = lane & 15, lk = lane >> 4;
  double tr[NFAM][KS];
#pragma unroll
  for (int f = 0; f < NFAM; ++f)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) tr[f][ks] = tab[(size_t)f * K + (s0 + li) * N + 4 * ks + lk];
  const int count = *count_ptr;
  for (int base = blockIdx.x * GPW; base < count; base += gridDim.x * GPW) {
    const int node = base + g;
    const bool live = node < count;
    double e = 0.0, s = 0.0;
    const JobDev* jb = nullptr;
    if (live) {
      jb = &jobs[lv.job[node]];
      const int bx = lv.x0[node], by = lv.y0[node];
#pragma unroll
      for (int i0 = 0; i0 < K; i0 += TPN) {
        const int i = i0 + tn;
        const int y = i / N, x = i % N;
        const double v = job_pixel(*jb, by + y, bx + x);
        sY[g][sw<N>(y, x)] = v;
        e = fma(v, v, e);
        s += v;
      }
    }
    e = wave_sum_f64(e);
    s = wave_sum_f64(s);
    if (lane == 0) {
      sRed[g][wn][0] = e;
      sRed[g][wn][1] = s;
    }
    __syncthreads();   // sY, sRed ready
    if (live) {
      e = sRed[g][0][0];
      s = sRed[g][0][1];
#pragma unroll
      for (int q = 1; q < WPN; ++q) {
        e += sRed[g][q][0];
        s += sRed[g][q][1];
      }
      if (tn == 0) {
        lv.e[node] = e;
        lv.t[node] = 0;
        uint8_t st = ST_RUN;
        if (e < jb->eps2[lg])
          st = ST_ACC;
        else if (jb->k[lg] <= 0)
          st = ST_SPARSE;
        lv.st[node] = st;
      }
    }
    double* cn = cbuf + (size_t)node * M;
#pragma unroll
    for (int f = 0; f < NFAM; ++f) {
      // Z^T[x][p] = sum_y Y[y][x] T_f[p][y], p in this wave's strip
      d4 acc[T];
#pragma unroll
      for (int tx = 0; tx < T; ++tx) acc[tx] = d4{0.0, 0.0, 0.0, 0.0};
      if (live) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int k = 4 * ks + lk;
#pragma unroll
          for (int tx = 0; tx < T; ++tx) acc[tx] = mfma64(sY[g][sw<N>(k, 16 * tx + li)], tr[f][ks], acc[tx]);
        }
      }
      __syncthreads();   // the previous family's second product is done with sZt
      if (live) {
#pragma unroll
        for (int tx = 0; tx < T; ++tx)
#pragma unroll
          for (int r = 0; r < 4; ++r) sZt[g][sw<N>(16 * tx + lk + 4 * r, s0 + li)] = acc[tx][r];
      }
      __syncthreads();   // Z^T complete
      if (live) {
        // C^T[q][p] = sum_x T_f[q][x] Z^T[x][p], q in this wave's strip
#pragma unroll
        for (int tp = 0; tp < T; ++tp) acc[tp] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int k = 4 * ks + lk;
#pragma unroll
          for (int tp = 0; tp < T; ++tp) acc[tp] = mfma64(tr[f][ks], sZt[g][sw<N>(k, 16 * tp + li)], acc[tp]);
        }
        // atom f K + q N + p; the constant atom (p = q = 0) is exactly 1/N
#pragma unroll
        for (int tp = 0; tp < T; ++tp)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int q = s0 + lk + 4 * r, pp = 16 * tp + li;
            cn[f * K + q * N + pp] = (q == 0 && pp == 0) ? s / N : acc[tp][r];
          }
      }
    }
    // The next round's gather writes sY: every wave has passed the barriers
    // after its last read of sY (first product of the last family).
  }
}

// Geometry of the whole-node pursuit: one wave per node for N <= 32, four for
// N = 64, each owning 16-wide strips of the row index q (SW of them) with the
// correlations in the matrix cores' output layout: value 4 (s T + tp) + r of
// a lane is atom (q = 16 (WPN s.. + s) + lane / 16 + 4 r, p = 16 tp + lane % 16).
template <int N, int NFAM>
struct PurGeo {
  static constexpr int K = N * N;
  static constexpr int M = NFAM * K;
  static constexpr int WPN = N == 64 ? 4 : 1;      // waves per node
  static constexpr int NPW = 4 / WPN;              // nodes per workgroup
  static constexpr int T = N / 16;
  static constexpr int SW = T / WPN;               // strips per wave
  static constexpr int AF = 4 * SW * T;            // correlations per lane and family
  static constexpr int G = AF / 4 * NFAM;          // groups of four
  static constexpr int KS = N / 4;
};
// CNT pixels of column x, rows y0, y0 + dy, ..
template <int CNT>
__device__ inline void job_column(const JobDev& jb, int y0, int dy, int x, double (&v)[CNT]) {
  const int xx = x < jb.w ? x : jb.w - 1;
  int64_t at[CNT];
#pragma unroll
  for (int i = 0; i < CNT; ++i) {
    const int y = y0 + i * dy;
    at[i] = (int64_t)(y < jb.h ? y : jb.h - 1) * jb.row_stride + xx;
  }
  if (jb.dtype == AQMP_F64) {
    const gmem_f64* p = (const gmem_f64*)jb.img;
#pragma unroll
    for (int i = 0; i < CNT; ++i) v[i] = p[at[i]];
  } else {
    const gmem_f32* p = (const gmem_f32*)jb.img;
#pragma unroll
    for (int i = 0; i < CNT; ++i) v[i] = (double)p[at[i]];
  }
}
template <int A>
struct DVec;
template <>
struct DVec<16> {
  typedef double type __attribute__((ext_vector_type(16)));
};
template <>
struct DVec<4> {
  typedef double type __attribute__((ext_vector_type(4)));
};

// Larger of |a| and b >= 0 (no quieting of NaNs first).  A matrix-core result
// may not go in: the compiler adds no wait states before inline assembly that
// reads one.  (It does before a lane exchange that reads the result of inline
// assembly; the one here does not rely on that.)
__device__ inline double max_abs(double a, double b) {
  double r;
  __asm__("v_max_f64 %0, |%1|, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// Best atom of a wave: largest |c|, lowest atom index among equal
// magnitudes; the result is uniform across the wave.  |c| is non-negative,
// so its bit pattern orders like its value.
__device__ inline void wave_best(double bc, int bi, double& wbc, int& wbi) {
  const unsigned long long mb = (unsigned long long)__double_as_longlong(fabs(bc));
  const unsigned long long m = wave_max_u64(mb);
  unsigned long long ball = __ballot(mb == m);
  int best = 0x7fffffff, L = 0;
  while (ball) {
    const int l = __builtin_ctzll(ball);
    const int cand = __builtin_amdgcn_readlane(bi, l);
    if (cand < best) {
      best = cand;
      L = l;
    }
    ball &= ball - 1;
  }
  const long long v = __double_as_longlong(bc);
  const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffffLL), L);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), L);
  wbc = __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
  wbi = best;
}

// Largest |v[j]| of a register array and its position, lowest j among equal
// magnitudes (pairwise tree: the left operand always holds lower positions).
template <int A>
__device__ inline void lane_best(const double (&c)[A], double& bc, int& bj) {
  double v[A];
  int ix[A];
#pragma unroll
  for (int j = 0; j < A; ++j) {
    v[j] = c[j];
    ix[j] = j;
  }
#pragma unroll
  for (int w = 1; w < A; w *= 2)
#pragma unroll
    for (int i = 0; i + w < A; i += 2 * w) {
      const bool take = fabs(v[i + w]) > fabs(v[i]);
      v[i] = take ? v[i + w] : v[i];
      ix[i] = take ? ix[i + w] : ix[i];
    }
  bc = v[0];
  bj = ix[0];
}

// The whole pursuit of every node: gather, ||y||^2, first stop test, the
// initial correlations (the two products of k_gram_init, in its order), then
// the steps, everything in registers and LDS.  Z^T takes the place of the
// pixels, so that N = 64 fits two workgroups to a CU beside X.
//
// What bounds it: N = 64 the FP64 products (2.1 MFLOP a node, 82 us for 3 072
// nodes at the matrix cores' FP64 rate) beside the chain of a node's steps,
// smaller blocks that chain.  Three 2048 x 2048 planes, N = 64 / 32 / 16:
// 261 / 95 / 77 us; 323 / 123 / 82 us with the correlations through memory
// (200 MB at N = 64) between two launches and a compare and three selects per
// correlation for the arg-max.
template <int N, int NFAM>
__global__ __launch_bounds__(256, 2) void k_gram_pursuit(const JobDev* __restrict__ jobs, LevelDev lv,
                                                         const int32_t* __restrict__ count_ptr,
                                                         int32_t* __restrict__ queue, int32_t lg,
                                                         const double* __restrict__ tab,
                                                         const double* __restrict__ xg) {
  using P = PurGeo<N, NFAM>;
  constexpr int K = P::K, WPN = P::WPN, NPW = P::NPW, T = P::T, SW = P::SW, AF = P::AF, G = P::G, KS = P::KS;
  constexpr int NX = NFAM == 2 ? N : 1;
  using CV = typename DVec<AF>::type;
  __shared__ double sX[NX][NX + 1];       // X[p][p'] = <T_0[p], T_1[p']>
  __shared__ double sYZ[NPW][K];          // pixels, then Z^T of a family
  __shared__ double sRed[4][2];
  __shared__ __attribute__((aligned(16))) double sBc[2][4];   // per-wave best, double-buffered (N = 64)
  __shared__ __attribute__((aligned(16))) int sBi[2][4];
  __shared__ int sNode[2][4];             // next node, double-buffered
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = WPN > 1 ? wv : 0, grp = WPN > 1 ? 0 : wv;
  const int li = lane & 15, lk = lane >> 4;
  double* yz = sYZ[grp];
  auto sync = [&]() {
    if constexpr (WPN > 1) __syncthreads();
    else wave_sync();
  };
  double tr[NFAM][SW][KS];
#pragma unroll
  for (int f = 0; f < NFAM; ++f)
#pragma unroll
    for (int s = 0; s < SW; ++s)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) tr[f][s][ks] = tab[(size_t)f * K + (16 * (wn * SW + s) + li) * N + 4 * ks + lk];
  if constexpr (NFAM == 2)
    for (int i = tid; i < K; i += 256) sX[i / N][i % N] = xg[i];
  __syncthreads();
  const int count = *count_ptr;
  const int q0 = (int)gridDim.x * NPW, qk = (int)blockIdx.x % kQueues;
  int ph = 0, np = 0;
  int node = (int)blockIdx.x * NPW + grp;
  while (node < count) {
    const int jidx = lv.job[node];
    const int bx = lv.x0[node], by = lv.y0[node];
    const JobDev jb = jobs[jidx];
    const double eps2 = jobs[jidx].eps2[lg];
    const int kmax = __builtin_amdgcn_readfirstlane(jobs[jidx].k[lg]);
    // ---- gather; ||y||^2 and the sum in k_gram_init's lanes and order ----
    double e, sum;
    if constexpr (N == 32) {
      double ev[2] = {0.0, 0.0}, sv[2] = {0.0, 0.0};   // its two waves
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        double pv[K / 128];
        job_column(jb, by + (64 * v + lane) / N, 128 / N, bx + lane % N, pv);
#pragma unroll
        for (int i0 = 0; i0 < K / 128; ++i0) {
          const int i = 128 * i0 + 64 * v + lane;
          yz[sw<N>(i / N, i % N)] = pv[i0];
          ev[v] = fma(pv[i0], pv[i0], ev[v]);
          sv[v] += pv[i0];
        }
        ev[v] = wave_sum_f64(ev[v]);
        sv[v] = wave_sum_f64(sv[v]);
      }
      e = ev[0] + ev[1];
      sum = sv[0] + sv[1];
    } else {
      constexpr int TPN = 64 * WPN;
      const int tn = WPN > 1 ? tid : lane;
      double ee = 0.0, ss = 0.0, pv[K / TPN];
      job_column(jb, by + tn / N, TPN / N, bx + tn % N, pv);
#pragma unroll
      for (int i0 = 0; i0 < K / TPN; ++i0) {
        const int i = TPN * i0 + tn;
        yz[sw<N>(i / N, i % N)] = pv[i0];
        ee = fma(pv[i0], pv[i0], ee);
        ss += pv[i0];
      }
      e = wave_sum_f64(ee);
      sum = wave_sum_f64(ss);
      if constexpr (WPN > 1) {
        if (lane == 0) {
          sRed[wv][0] = e;
          sRed[wv][1] = sum;
        }
      }
    }
    sync();
    if constexpr (WPN > 1) {
      e = sRed[0][0];
      sum = sRed[0][1];
#pragma unroll
      for (int q = 1; q < WPN; ++q) {
        e += sRed[q][0];
        sum += sRed[q][1];
      }
    }
    uint8_t st = ST_RUN;
    if (e < eps2)
      st = ST_ACC;
    else if (kmax <= 0)
      st = ST_SPARSE;
    CV c[NFAM];
    if (st == ST_RUN) {
      // Z^T[x][p] = sum_y Y[y][x] T_f[p][y], p in the wave's strips
      d4 z[NFAM][SW][T];
#pragma unroll
      for (int f = 0; f < NFAM; ++f)
#pragma unroll
        for (int s = 0; s < SW; ++s)
#pragma unroll
          for (int tx = 0; tx < T; ++tx) z[f][s][tx] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int tx = 0; tx < T; ++tx) {
          const double yv = yz[sw<N>(4 * ks + lk, 16 * tx + li)];
#pragma unroll
          for (int f = 0; f < NFAM; ++f)
#pragma unroll
            for (int s = 0; s < SW; ++s) z[f][s][tx] = mfma64(yv, tr[f][s][ks], z[f][s][tx]);
        }
#pragma unroll
      for (int f = 0; f < NFAM; ++f) {
        sync();   // the pixels, or the other family's Z^T, are read
#pragma unroll
        for (int s = 0; s < SW; ++s)
#pragma unroll
          for (int tx = 0; tx < T; ++tx)
#pragma unroll
            for (int r = 0; r < 4; ++r) yz[sw<N>(16 * tx + lk + 4 * r, 16 * (wn * SW + s) + li)] = z[f][s][tx][r];
        sync();
        // C^T[q][p] = sum_x T_f[q][x] Z^T[x][p], q in the wave's strips
        d4 a[SW][T];
#pragma unroll
        for (int s = 0; s < SW; ++s)
#pragma unroll
          for (int tp = 0; tp < T; ++tp) a[s][tp] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int tp = 0; tp < T; ++tp) {
            const double zv = yz[sw<N>(4 * ks + lk, 16 * tp + li)];
#pragma unroll
            for (int s = 0; s < SW; ++s) a[s][tp] = mfma64(tr[f][s][ks], zv, a[s][tp]);
          }
#pragma unroll
        for (int j = 0; j < AF; ++j)   // (an ordinary instruction between the matrix cores and max_abs)
          c[f][j] = __builtin_canonicalize(a[j / (4 * T)][(j >> 2) % T][j & 3]);
        // the constant atom (p = q = 0) is exactly 1/N
        if (wn == 0 && lane == 0) c[f][0] = sum / N;
      }
    }
    // The largest |c| is found by FP64 maxima; undefined pixels (or a norm
    // that overflows) by the order of the bits, where a NaN is the largest.
    const bool odd = !(e < __builtin_inf());
    constexpr int V = NFAM * AF;
    int t = 0;
    int rec_i = 0;
    double rec_c = 0.0;
    const size_t rec0 = (size_t)node * lv.kmax;
    auto atom_of = [&](int f, int j, int w, int l) -> int {
      return f * K + (16 * (w * SW + j / (4 * T)) + (l >> 4) + 4 * (j & 3)) * N + 16 * ((j >> 2) % T) + (l & 15);
    };
    while (st == ST_RUN) {
      // ---- the wave's arg-max |c|, lowest atom index on ties ----
      if constexpr (NFAM == 2) {
        // the second family's constant atom equals the first's, which wins the
        // tie (and with which it goes to zero)
        if (wn == 0 && lane == 0) c[1][0] = 0.0;
      }
      int bi = 0x7fffffff, at = 0, L = 0;            // atom; its place f AF + j and lane
      uint32_t is = 0u;                              // bit V - 1 - j: value j is the wave's largest
      bool one = !odd;
      if (!odd) {
        double m0 = 0.0, m1 = 0.0;
#pragma unroll
        for (int f = 0; f < NFAM; ++f)
#pragma unroll
          for (int j = 0; j < AF; j += 2) {
            m0 = max_abs(c[f][j], m0);
            m1 = max_abs(c[f][j + 1], m1);
          }
        // (an ordinary instruction between max_abs and the lane exchanges)
        const double m = wave_max_f64(__builtin_canonicalize(max_abs(m0, m1)));
        // the sign of |c| - m, two instructions per value: bit V - 1 - j is 0
        // where value j is the largest
        uint32_t less = ~0u;
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const double d = fabs(c[j / AF][j % AF]) - m;
          less = __builtin_amdgcn_alignbit(less, (uint32_t)((unsigned long long)__double_as_longlong(d) >> 32), 31);
        }
        is = ~less;
        const unsigned long long hit = __ballot(is != 0u);
        L = hit ? __builtin_ctzll(hit) : 0;
        const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)is, L);
        one = __popcll(hit) == 1 && __popc(bits) == 1;
        at = V - 1 - (bits ? __builtin_ctz(bits) : 0);
        bi = atom_of(at / AF, at % AF, wn, L);
      }
      if (!one) {
        // Ties (Haar atoms on replicated rows or binary planes tie at most
        // steps), or undefined values: the lowest atom of those that are the
        // largest, undefined values by their bits.
        int best = 0x7fffffff;
        if (!odd) {
          for (uint32_t u = is; __ballot(u != 0u) != 0ull; u &= u - 1u) {
            const int j = V - 1 - (u ? __builtin_ctz(u) : 0);
            const int a = atom_of(j / AF, j % AF, wn, lane);
            best = u != 0u && a < best ? a : best;
          }
        } else {
          unsigned long long mb = 0ull;
#pragma unroll
          for (int f = 0; f < NFAM; ++f)
#pragma unroll 1
            for (int j = 0; j < AF; ++j) {
              const unsigned long long u = (unsigned long long)__double_as_longlong(fabs(c[f][j]));
              mb = u > mb ? u : mb;
            }
          const unsigned long long m = wave_max_u64(mb);
#pragma unroll
          for (int f = 0; f < NFAM; ++f)
#pragma unroll 1
            for (int j = 0; j < AF; ++j) {
              const int a = atom_of(f, j, wn, lane);
              if ((unsigned long long)__double_as_longlong(fabs(c[f][j])) == m && a < best) best = a;
            }
        }
        bi = wave_min_i32(best);
        const int q = (bi % K) / N, p = bi % N;
        at = bi / K * AF + 4 * (((q >> 4) % SW) * T + (p >> 4)) + ((q & 15) >> 2);
        L = (q & 3) * 16 + (p & 15);
      }
      at = __builtin_amdgcn_readfirstlane(at);
      L = __builtin_amdgcn_readfirstlane(L);
      double bc;
      {
        double v;
        if (NFAM == 1 || at < AF) v = c[0][at % AF];
        else v = c[NFAM - 1][at % AF];
        const unsigned long long u = (unsigned long long)__double_as_longlong(v);
        const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, L);
        const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), L);
        bc = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
      }
      int ow = 0;                                    // the wave that holds the atom
      if constexpr (WPN > 1) {
        if (lane == 0) {
          sBc[ph][wv] = bc;
          sBi[ph][wv] = bi;
        }
        __syncthreads();
        const double2 b01 = *(const double2*)&sBc[ph][0], b23 = *(const double2*)&sBc[ph][2];
        const int4 bj = *(const int4*)&sBi[ph][0];
        const double wb[4] = {b01.x, b01.y, b23.x, b23.y};
        const int wi[4] = {bj.x, bj.y, bj.z, bj.w};
        bc = wb[0];
        bi = wi[0];
#pragma unroll
        for (int q = 1; q < WPN; ++q) {
          const bool take = fabs(wb[q]) > fabs(bc) || (fabs(wb[q]) == fabs(bc) && wi[q] < bi);
          bc = take ? wb[q] : bc;
          bi = take ? wi[q] : bi;
        }
        bi = __builtin_amdgcn_readfirstlane(bi);
        ow = (bi % K) / N / (16 * SW);
        ph ^= 1;
      }
      if (bc == 0.0) {
        st = ST_ZERO;
        break;
      }
      if (lane == t % 64) {
        rec_i = bi;
        rec_c = bc;
      }
      // c_a <- c_a - c_i <phi_a, phi_i>: zero for the atom itself, nothing for
      // the rest of its family, X[p_a][p_i] X[q_a][q_i] (or its transpose)
      // for the other family, exact for the constant atoms.
      const int pi = bi % N, qi = (bi % K) / N;
      const bool first = NFAM == 1 || bi < K;
      const bool own = (WPN == 1 || ow == wn) && lane == L;
      if constexpr (NFAM == 2 && N == 16) {
        // Four values of a family: a branch on it.  All of 100 steps, 16 / 4 096
        // nodes: 74 / 143 us; without it, as below, 81 / 164.
        auto step = [&](CV& same, CV& other, auto x) {
          const double bv = -bc * x(pi, li);
          double xq[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) xq[r] = x(qi, lk + 4 * r);
#pragma unroll
          for (int j = 0; j < AF; ++j) {
            same[j] = own && j == at % AF ? 0.0 : same[j];
            other[j] = fma(bv, xq[j], other[j]);
          }
        };
        if (first) step(c[0], c[1], [&](int i, int k) { return sX[i][k]; });
        else step(c[1], c[0], [&](int i, int k) { return sX[k][i]; });
      } else {
#pragma unroll
        for (int f = 0; f < NFAM; ++f) {
          const double v = c[f][at % AF];
          c[f][at % AF] = own && first == (f == 0) ? 0.0 : v;
        }
      }
      if constexpr (NFAM == 2 && N > 16) {
        // (no branch on the family, whose joins copied all of them: the atom's
        // own family takes zero times the products)
        double bv[T], xq[SW][4];
#pragma unroll
        for (int tp = 0; tp < T; ++tp) bv[tp] = -bc * (first ? sX[pi][16 * tp + li] : sX[16 * tp + li][pi]);
#pragma unroll
        for (int s = 0; s < SW; ++s)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int q = 16 * (wn * SW + s) + lk + 4 * r;
            xq[s][r] = first ? sX[qi][q] : sX[q][qi];
          }
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          double bf[T];
#pragma unroll
          for (int tp = 0; tp < T; ++tp) bf[tp] = first == (f == 1) ? bv[tp] : 0.0;
#pragma unroll
          for (int j = 0; j < AF; ++j) c[f][j] = fma(bf[(j >> 2) % T], xq[j / (4 * T)][j & 3], c[f][j]);
        }
      }
      e = fma(-bc, bc, e);
      ++t;
      if (t % 64 == 0 && wn == 0) {
        lv.rec_idx[rec0 + (t - 64) + lane] = rec_i;
        lv.rec_coef[rec0 + (t - 64) + lane] = rec_c;
      }
      if (e < eps2)
        st = ST_ACC;
      else if (t >= kmax)
        st = ST_SPARSE;
    }
    if (WPN > 1 ? tid == 0 : lane == 0) sNode[np][grp] = q0 + atomicAdd(queue + qk * kQueuePad, 1) * kQueues + qk;
    if (wn == 0) {
      if (lane < t % 64) {
        lv.rec_idx[rec0 + (t - t % 64) + lane] = rec_i;
        lv.rec_coef[rec0 + (t - t % 64) + lane] = rec_c;
      }
      if (lane == 0) {
        lv.e[node] = e;
        lv.t[node] = t;
        lv.st[node] = st;
      }
    }
    sync();   // the next node; yz is read
    node = __builtin_amdgcn_readfirstlane(sNode[np][grp]);
    np ^= 1;
  }
}

// ---------------------------------------------------------------------------
// Small blocks.  N = 4, and few nodes of N = 8: K = N^2 lanes per node (a row
// of 16, or the wave), lane = pixel for the gather and lane = (p, q) for the
// atoms, one atom per family per lane.  The correlations come from the
// separable sum sum_y T_f[p][y] sum_x T_f[q][x] Y[y][x]; the pursuit then runs
// on the Gram updates as above.  Selection reductions are lane exchanges: the
// largest |c|, then the lowest atom index among the lanes holding it, then
// that lane's c.
// ---------------------------------------------------------------------------
__device__ inline double row_sum_f64(double d) {
  d += row_perm_f64<0xB1>(d);
  d += row_perm_f64<0x4E>(d);
  d += row_perm_f64<0x141>(d);
  d += row_perm_f64<0x140>(d);
  return d;
}

// The nodes node, node + step, .. of the lane's group; sT: T_f[p][y] at
// [f][p N + y]; ys: K doubles of the group's own; cross(f, p, q): <phi, phi'>
// of atom (f, p, q) with the lane's atom of the other family.
template <int N, int NFAM, class Cross>
__device__ inline void gram_pixels(const JobDev* __restrict__ jobs, const LevelDev& lv, int node, int step, int count,
                                   const double* sT, double* ys, Cross cross) {
  constexpr int K = N * N, lg = N == 4 ? 2 : 3;
  static_assert(K == 16 || K == 64, "a row of lanes or a wave");
  const int lt = (int)threadIdx.x % K;
  const int pa = lt % N, qa = lt / N;    // this lane's atoms f K + lt
  auto sum = [](double v) -> double {
    if constexpr (K == 64) return wave_sum_f64(v);
    else return row_sum_f64(v);
  };
  for (; node < count; node += step) {
    const JobDev& jb = jobs[lv.job[node]];
    const double eps2 = jb.eps2[lg];
    const int kmax = jb.k[lg];
    const double v = job_pixel(jb, lv.y0[node] + qa, lv.x0[node] + pa);   // pixel (lt / N, lt % N)
    ys[lt] = v;
    __builtin_amdgcn_wave_barrier();     // group-private: the wave's own writes are seen by its reads
    double e = sum(v * v);
    const double s = sum(v);
    uint8_t st = ST_RUN;
    if (e < eps2)
      st = ST_ACC;
    else if (kmax <= 0)
      st = ST_SPARSE;
    double c[NFAM];
#pragma unroll
    for (int f = 0; f < NFAM; ++f) {
      double acc = 0.0;
#pragma unroll 4
      for (int y = 0; y < N; ++y) {
        double u = 0.0;
#pragma unroll
        for (int x = 0; x < N; ++x) u = fma(sT[f * K + qa * N + x], ys[y * N + x], u);
        acc = fma(sT[f * K + pa * N + y], u, acc);
      }
      c[f] = lt == 0 ? s / N : acc;
    }
    __builtin_amdgcn_wave_barrier();     // ys is rewritten by the next node
    int t = 0, rec_i = 0;
    double rec_c = 0.0;
    const size_t rec0 = (size_t)node * lv.kmax;
    while (st == ST_RUN) {
      double bc = c[0];
      int bi = lt;
      if constexpr (NFAM == 2) {
        const bool take = fabs(c[1]) > fabs(bc);
        bc = take ? c[1] : bc;
        bi = take ? K + lt : bi;
      }
      const unsigned long long mb = (unsigned long long)__double_as_longlong(fabs(bc));
      unsigned long long m;
      if constexpr (K == 64) {
        m = wave_max_u64(mb);
        bi = wave_min_i32(mb == m ? bi : 0x7fffffff);
      } else {
        m = row_max_u64(mb);
        bi = row_min_i32(mb == m ? bi : 0x7fffffff);
      }
      if (m == 0ull) {
        st = ST_ZERO;
        break;
      }
      bc = sum((lt == bi % K) ? (bi >= K ? c[NFAM - 1] : c[0]) : 0.0);
      if (lt == t % K) {
        rec_i = bi;
        rec_c = bc;
      }
      const int fi = bi / K, pi = bi % N, qi = (bi % K) / N;
      // same family: only c_i changes (to zero); other family: X products
#pragma unroll
      for (int f = 0; f < NFAM; ++f) {
        if (f == fi)
          c[f] = (lt == bi % K) ? 0.0 : c[f];
        else if constexpr (NFAM == 2)
          c[f] = fma(-bc, cross(fi, pi, qi), c[f]);
      }
      e = fma(-bc, bc, e);
      ++t;
      if (t % K == 0) {
        lv.rec_idx[rec0 + (t - K) + lt] = rec_i;
        lv.rec_coef[rec0 + (t - K) + lt] = rec_c;
      }
      if (e < eps2)
        st = ST_ACC;
      else if (t >= kmax)
        st = ST_SPARSE;
    }
    if (lt < t % K) {
      lv.rec_idx[rec0 + (t - t % K) + lt] = rec_i;
      lv.rec_coef[rec0 + (t - t % K) + lt] = rec_c;
    }
    if (lt == 0) {
      lv.e[node] = e;
      lv.t[node] = t;
      lv.st[node] = st;
    }
  }
}

template <int NFAM>
__global__ __launch_bounds__(256) void k_gram4(const JobDev* __restrict__ jobs, LevelDev lv,
                                               const int32_t* __restrict__ count_ptr, const double* __restrict__ tab,
                                               const double* __restrict__ xg) {
  constexpr int N = 4, K = N * N;
  constexpr int NG = 256 / K;            // nodes per workgroup
  constexpr int NX = NFAM == 2 ? N : 1;
  __shared__ double sT[NFAM][K];         // T_f[p][y] at [f][p N + y]
  __shared__ double sX[NX][NX + 1];      // X[p][p'] = <T_0[p], T_1[p']>
  __shared__ double sY[NG][K];           // the node's pixels (group-private)
  const int tid = threadIdx.x, grp = tid / K, pa = tid % N, qa = tid % K / N;
  for (int i = tid; i < NFAM * K; i += 256) (&sT[0][0])[i] = tab[i];
  if constexpr (NFAM == 2)
    for (int i = tid; i < K; i += 256) sX[i / N][i % N] = xg[i];
  __syncthreads();
  gram_pixels<N, NFAM>(jobs, lv, blockIdx.x * NG + grp, gridDim.x * NG, *count_ptr, &sT[0][0], sY[grp],
                       [&](int f, int p, int q) -> double {
                         return f ? sX[pa][p] * sX[qa][q] : sX[p][pa] * sX[q][qa];
                       });
}

// N = 8.  Up to kGram8Waves nodes: a wave each, a lane per pixel
// (gram_pixels).  More: four nodes per wave, 16 lanes each.
// Lane li of a node holds pixels
// (li / 2, 4 (li % 2) ..) and, of each family, atoms q = li / 2, p = 4 (li %
// 2) + r, r = 0..3, so that a reduction over a node is four row operations
// for all four nodes at once.  The sums and the updates are those of a lane per
// pixel, bit for bit.  A slot whose node has ended takes its next one from the
// queues.
// What bounds it: the instructions of a step (about 200 for four nodes; 130
// for one node with a lane per pixel).  11 152 nodes, 170 692 steps: 44 us,
// 74 us with a wave per node and a lane per pixel.
// The line between them, by the nodes that the level has: two waves per SIMD of
// the chip.  Two families, all of 57 steps / pursuits that end early (3 on
// average, at most 15), a wave per node against four to a wave: 1 024 nodes 53
// / 38 against 63 / 46 us, 2 048 60 / 38 against 64 / 45, 2 304 70 / 40 against
// 64 / 46, 4 096 92 / 45 against 65 / 47.
constexpr int kGram8Waves = 2048;
template <int NFAM>
__global__ __launch_bounds__(256) void k_gram8(const JobDev* __restrict__ jobs, LevelDev lv,
                                               const int32_t* __restrict__ count_ptr, int32_t* __restrict__ queue,
                                               const double* __restrict__ tab, const double* __restrict__ xg) {
  constexpr int N = 8, K = 64, LPS = 16, SN = 4, lg = 3;
  constexpr int YP = K + 2;               // doubles of a node's pixels (a node's on banks of its own)
  __shared__ __attribute__((aligned(16))) double sT[NFAM][N][N];    // T_f[p][y]
  __shared__ __attribute__((aligned(16))) double sTt[NFAM][N][N];   // and by [y][p]
  __shared__ __attribute__((aligned(16))) double sX[2][N][N];       // [f][p][p']: row p of family f against the other
  __shared__ __attribute__((aligned(16))) double sY[4][SN * YP];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < NFAM * K; i += 256) {
    const double v = tab[i];
    const int f = i / K, pp = i % K / N, y = i % N;
    sT[f][pp][y] = v;
    sTt[f][y][pp] = v;
  }
  if constexpr (NFAM == 2)
    if (tid < K) {
      const double v = xg[tid];
      sX[0][tid / N][tid % N] = v;
      sX[1][tid % N][tid / N] = v;
    }
  __syncthreads();
  const int count = *count_ptr;
  if (count <= kGram8Waves) {
    gram_pixels<N, NFAM>(jobs, lv, (int)blockIdx.x * 4 + wv, (int)gridDim.x * 4, count, &sT[0][0][0], sY[wv],
                         [&](int f, int p, int q) -> double { return sX[f][p][lane % N] * sX[f][q][lane / N]; });
    return;
  }
  const int slot = lane / LPS, li = lane % LPS, q = li >> 1, p0 = 4 * (li & 1);
  double* ys = sY[wv] + slot * YP;
  const int q0 = (int)gridDim.x * 4 * SN, qk = (int)blockIdx.x % kQueues;
  int node = ((int)blockIdx.x * 4 + wv) * SN + slot;
  bool dry = node >= count, run = false, load = !dry;
  int t = 0, kmax = 0, rec_i = 0;
  double rec_c = 0.0, e = 0.0, eps2 = 0.0;
  double c[NFAM][4];
#pragma unroll
  for (int f = 0; f < NFAM; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) c[f][r] = 0.0;
  auto slot_sum = [](double v) -> double {   // pixels in the order of their bits
    v += row_perm_f64<0xB1>(v);
    v += row_perm_f64<0x4E>(v);
    v += row_perm_f64<0x141>(v);
    v += row_perm_f64<0x128>(v);
    return v;
  };
  for (;;) {
    if (__ballot(load) != 0ull) {
      if (load) {
        const int jidx = lv.job[node];
        const int bx = lv.x0[node], by = lv.y0[node];
        const JobDev jl = jobs[jidx];
        eps2 = jobs[jidx].eps2[lg];
        kmax = jobs[jidx].k[lg];
        double v[4];
        job_pixels<4>(jl, by + q, bx + p0, v);
#pragma unroll
        for (int j = 0; j < 4; j += 2) *(double2*)&ys[q * N + p0 + j] = make_double2(v[j], v[j + 1]);
        // of each pair of squares one is rounded by itself: the odd pixels' in
        // the left half of a row, the even pixels' in the right one
        const bool rh = p0 != 0;
        const double a0 = rh ? v[1] : v[0], a1 = rh ? v[0] : v[1], a2 = rh ? v[3] : v[2], a3 = rh ? v[2] : v[3];
        e = slot_sum(fma(a0, a0, a1 * a1) + fma(a2, a2, a3 * a3));
        const double s = slot_sum((v[0] + v[1]) + (v[2] + v[3]));
        t = 0;
        uint8_t st = ST_RUN;
        if (e < eps2)
          st = ST_ACC;
        else if (kmax <= 0)
          st = ST_SPARSE;
        run = st == ST_RUN;
        if (!run && li == 0) {
          lv.e[node] = e;
          lv.t[node] = 0;
          lv.st[node] = st;
        }
        wave_sync();   // the node's pixels, read by its other lanes
        if (run) {
          // sum_y T_f[p][y] sum_x T_f[q][x] Y[y][x]
          double tq[NFAM][N];
#pragma unroll
          for (int f = 0; f < NFAM; ++f)
#pragma unroll
            for (int x = 0; x < N; ++x) tq[f][x] = sT[f][q][x];
#pragma unroll
          for (int f = 0; f < NFAM; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) c[f][r] = 0.0;
#pragma unroll 2
          for (int y = 0; y < N; ++y) {
            double px[N];
#pragma unroll
            for (int x = 0; x < N; ++x) px[x] = ys[y * N + x];
#pragma unroll
            for (int f = 0; f < NFAM; ++f) {
              double u = 0.0;
#pragma unroll
              for (int x = 0; x < N; ++x) u = fma(tq[f][x], px[x], u);
#pragma unroll
              for (int r = 0; r < 4; ++r) c[f][r] = fma(sTt[f][y][p0 + r], u, c[f][r]);
            }
          }
          if (li == 0)
#pragma unroll
            for (int f = 0; f < NFAM; ++f) c[f][0] = s / N;
        }
        wave_sync();   // read before another node's pixels come
      }
    }
    if (__ballot(run) != 0ull) {
      // the larger of a lane's two families (the first on a tie), then the
      // largest by bits, the lowest atom among equals
      double bc[4];
      int bf[4];
      unsigned long long mb = 0ull;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        bc[r] = c[0][r];
        bf[r] = 0;
        if constexpr (NFAM == 2) {
          const bool take = fabs(c[1][r]) > fabs(c[0][r]);
          bc[r] = take ? c[1][r] : c[0][r];
          bf[r] = take ? K : 0;
        }
        const unsigned long long u = (unsigned long long)__double_as_longlong(fabs(bc[r]));
        mb = u > mb ? u : mb;
      }
      const unsigned long long m = row_max_u64(mb);
      int bi = 0x7fffffff;
#pragma unroll
      for (int r = 3; r >= 0; --r) {
        const int a = bf[r] + q * N + p0 + r;
        if ((unsigned long long)__double_as_longlong(fabs(bc[r])) == m && a < bi) bi = a;
      }
      bi = row_min_i32(bi);
      const bool zero = m == 0ull;
      const int fi = NFAM == 2 && bi >= K ? 1 : 0, pi = bi % N, qi = bi % K / N;
      const bool mine = qi == q && (pi & 4) == p0;
      double v = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) v = mine && (pi & 3) == r ? (fi ? c[NFAM - 1][r] : c[0][r]) : v;
      const double b = slot_sum(v);
      // same family: only the atom's own changes (to zero); the other: X products
      double g[4] = {0.0, 0.0, 0.0, 0.0};
      if constexpr (NFAM == 2) {
        const double xq = sX[fi][qi & 7][q];
        const double2 x0 = *(const double2*)&sX[fi][pi][p0], x1 = *(const double2*)&sX[fi][pi][p0 + 2];
        g[0] = x0.x * xq;
        g[1] = x0.y * xq;
        g[2] = x1.x * xq;
        g[3] = x1.y * xq;
      }
      if (run && !zero) {
        if (li == (t & 15)) {
          rec_i = bi;
          rec_c = b;
        }
#pragma unroll
        for (int f = 0; f < NFAM; ++f) {
          const double nb = fi == f ? 0.0 : -b;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double w = c[f][r];
            if constexpr (NFAM == 2) w = fma(nb, g[r], w);
            c[f][r] = fi == f && mine && (pi & 3) == r ? 0.0 : w;
          }
        }
        e = fma(-b, b, e);
        ++t;
      }
      if (run) {
        uint8_t st = ST_RUN;
        if (zero)
          st = ST_ZERO;
        else if (e < eps2)
          st = ST_ACC;
        else if (t >= kmax)
          st = ST_SPARSE;
        // records of the last up to 16 steps
        const int base = zero ? t & ~15 : (t - 1) & ~15;
        if ((st != ST_RUN || t - base == 16) && li < t - base) {
          const size_t rs = (size_t)node * lv.kmax + base + li;
          lv.rec_idx[rs] = rec_i;
          lv.rec_coef[rs] = rec_c;
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
      int ahead = 0;
      if (!run && !dry && li == 0) ahead = atomicAdd(queue + qk * kQueuePad, 1);
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

// ---------------------------------------------------------------------------
// Orthogonal Matching Pursuit (the solver of the authors' implementation,
// Section 2.2): the selection of MP, then every selected coefficient re-fit by
// least squares, x_S = argmin ||y - D_S x||.  Computed in correlation space
// with the same Gram structure:
//   * L = the inverse of the Cholesky factor of the selected atoms' Gram
//     matrix G_SS (lower triangular, in LDS), one new row per step: with
//     g = G_{S,i} and w = L g, d = sqrt(1 - w.w), the row is (-w^T L, 1) / d;
//   * z = L D_S^T y grows by z_t = (<y, phi_i> - w.z) / d, so
//     ||r||^2 = ||y||^2 - ||z||^2 drops by z_t^2, and x_S = L^T z;
//   * c = D^T r = c0 - G_{:,S} x_S: within a family the Gram column is a
//     Kronecker delta (the selected atoms' own correlations are exactly zero,
//     r being orthogonal to them), across families the X products.
// One workgroup per node at every N (the per-step solves are small and
// serial), nodes handed out from queues.  c0 = D^T y comes from
// k_gram_init for N >= 16 and is computed here for N <= 8.
// What bounds it: the chain of a step (5 300 cycles at N = 8: arg-max 640,
// Gram entries and w 1 170, root, quotients and the new row 1 650, refresh
// 1 600), of which a CU holds as many as the factors leave room for.  Three
// 1024 x 1024 planes, k = 32, N = 64 / 32 / 16 / 8: 187 / 145 / 135 / 129 us;
// 204 / 212 / 168 / 176 us with loops over single selections, each waiting
// for its loads, and thousands of workgroups starting on one counter (20 to
// 25 us of every node's start).
// ---------------------------------------------------------------------------
template <int N, int NFAM>
struct OmpGeo {
  static constexpr int K = N * N;
  static constexpr int M = NFAM * K;
  static constexpr bool SMALL = N <= 8;                // K <= 64: one wave, lane k holds atom (f, k) of each family, c0 computed here
  // threads per node: one wave at N <= 16 (its workgroup barriers are the
  // wave's own ordering), two waves at N = 32, eight at N = 64 (two 16 x 16
  // tiles per wave and family at either)
  static constexpr int NT = N <= 16 ? 64 : (N == 32 ? 128 : 512);
  // N >= 16 (MF): a family's N x N grid of (p, q) is cut into 16 x 16 tiles,
  // TPW consecutive tiles per wave; a lane holds, per tile, the four atoms of
  // the FP64 MFMA output layout: p = 16 tp + lane / 16 + 4 r,
  // q = 16 tq + lane % 16, as j = f AF + 4 i + r, so the cross-family refresh
  // is a rank-4 MFMA update per four selected atoms.  The atom index grows
  // with j, so the per-thread arg-max keeps the lowest index on ties.
  static constexpr bool MF = !SMALL;
  static constexpr int NT16 = N / 16;                  // tiles per row of a family's grid
  static constexpr int TPW = MF ? NT16 * NT16 / (NT / 64) : 1;   // tiles per wave per family
  static constexpr int AF = MF ? 4 * TPW : 1;          // atoms per thread per family
  static constexpr int APT = SMALL ? NFAM : NFAM * AF;
  // a wave's tiles cover the grid once and lie in one tile row (so that the
  // atom index grows with j); at most eight waves (the per-wave best slots)
  static_assert(!MF || (TPW * (NT / 64) == NT16 * NT16 && NT16 % TPW == 0), "tile split");
  static_assert(NT <= 512, "per-wave slots");
  __device__ static int atom(int tid, int j) {
    if constexpr (SMALL) return tid < K ? j * K + tid : M;   // lanes past K hold no atom
    const int f = j / AF, rem = j % AF, i = rem / 4, r = rem % 4, l = tid & 63;
    const int t = (tid >> 6) * TPW + i, tp = t / NT16, tq = t % NT16;
    return f * K + (16 * tq + (l & 15)) * N + 16 * tp + (l >> 4) + 4 * r;
  }
  __device__ static int owner(int a) {
    if constexpr (SMALL) return a % K;
    const int q = (a % K) / N, p = a % N, t = (p / 16) * NT16 + q / 16;
    return 64 * (t / TPW) + 16 * ((p % 16) % 4) + q % 16;
  }
  __device__ static int slot(int a) {
    if constexpr (SMALL) return a / K;
    const int q = (a % K) / N, p = a % N, t = (p / 16) * NT16 + q / 16;
    return (a / K) * AF + 4 * (t % TPW) + (p % 16) / 4;
  }
};

template <int N, int NFAM>
__global__ __launch_bounds__((OmpGeo<N, NFAM>::NT)) void k_omp(const JobDev* __restrict__ jobs, LevelDev lv,
                                             const int32_t* __restrict__ count_ptr, int32_t* queue, int32_t lg,
                                             const double* __restrict__ tab, const double* __restrict__ xg,
                                             const double* __restrict__ cbuf, int k8) {
  using G = OmpGeo<N, NFAM>;
  constexpr int K = G::K, M = G::M, APT = G::APT, AF = G::AF;
  constexpr bool SMALL = G::SMALL;
  constexpr int KC = kOmpMaxAtoms;
  constexpr int NX = NFAM == 2 ? N : 1;
  __shared__ double sX[NX][NX + 1];                    // X[p][p'] = <T_0[p], T_1[p']>
  __shared__ double sT[SMALL ? NFAM : 1][SMALL ? K : 1];
  __shared__ double sY[SMALL ? K : 1];
  // L = chol(G_SS)^-1, lower triangular, k8 rows of k8 + 1 doubles, sized at
  // launch by the largest k of the level, rounded up to eights (smaller k:
  // more workgroups per CU).  Rows are zero past the diagonal, and rows not
  // written yet hold finite values, so that its products run over whole
  // blocks of eight, their loads in flight together: the terms past the end
  // are exact zeros.
  extern __shared__ double sLdyn[];
  const int ldl = k8 + 1;
  __shared__ int sS[KC];                               // selected atoms in order
  __shared__ double sXc[KC], sG[KC], sW[KC];           // x_S, g, w
  // the selected atoms split by family, in selection order: p | q << 8 and x
  // (zeros behind the last: the refresh takes both in eights)
  __shared__ int sPQ[NFAM][KC + 8];
  __shared__ double sXF[NFAM][KC + 8];
  __shared__ int sNF[NFAM];
  __shared__ double sBc[2][8];                         // per-wave best c
  __shared__ int sBi[2][8];
  __shared__ double sScal[2];                          // dependence flag, new ||r||^2
  __shared__ double sRed[2];
  __shared__ int sNode[2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if constexpr (NFAM == 2)
    for (int i = tid; i < K; i += G::NT) sX[i / N][i % N] = xg[i];
  if constexpr (SMALL)
    for (int i = tid; i < NFAM * K; i += G::NT) (&sT[0][0])[i] = tab[i];
  for (int i = tid; i < k8 * ldl; i += G::NT) sLdyn[i] = 0.0;
  __syncthreads();
  const int count = *count_ptr;
  const int pa = tid % N;                              // p of the thread's atom (N <= 8)
  int ph = 0, np = 0;
  // The first nodes are dealt out in order, the others by the queues (see
  // k_pursuit_sep).
  const int qk = (int)blockIdx.x % kQueues;
  int node = (int)blockIdx.x;
  for (; node < count; node = sNode[np], np ^= 1) {
    if constexpr (NFAM == 2)
      for (int i = tid; i < NFAM * (KC + 8); i += G::NT) {
        (&sPQ[0][0])[i] = 0;
        (&sXF[0][0])[i] = 0.0;
      }
    __syncthreads();   // the lists are the wave's that fills them
    const JobDev& jb = jobs[lv.job[node]];
    const double eps2 = jb.eps2[lg];
    const int kmax = jb.k[lg];
    double e;
    uint8_t st;
    // c: the current correlations <r, phi_a> of the thread's atoms.  Small
    // blocks recompute them from c0 = D^T y each step; larger ones update
    // them in place (see the refresh).
    double c0[SMALL ? APT : 1], c[APT];
    if constexpr (SMALL) {
      // gather (pixel k in thread k), ||y||^2, sum y, first stop test, c0
      double v = 0.0;
      if (tid < K) {
        v = job_pixel(jb, lv.y0[node] + tid / N, lv.x0[node] + tid % N);
        sY[tid] = v;
      }
      if (wv == 0) {
        const double ee = wave_sum_f64(v * v), ss = wave_sum_f64(v);
        if (lane == 0) {
          sRed[0] = ee;
          sRed[1] = ss;
        }
      }
      __syncthreads();
      e = sRed[0];
      const double ssum = sRed[1];
      st = e < eps2 ? ST_ACC : (kmax <= 0 ? ST_SPARSE : ST_RUN);
#pragma unroll
      for (int f = 0; f < APT; ++f) {   // the lane's atom (f, p = tid % N, q = tid / N)
        double acc = 0.0;
        if (tid < K) {
          const int q = tid / N;
#pragma unroll
          for (int y = 0; y < N; ++y) {
            double u = 0.0;
#pragma unroll
            for (int x = 0; x < N; ++x) u = fma(sT[f][q * N + x], sY[y * N + x], u);
            acc = fma(sT[f][pa * N + y], u, acc);
          }
          if (tid == 0) acc = ssum / N;
        }
        c0[f] = acc;
        c[f] = acc;
      }
    } else {
      e = lv.e[node];
      st = lv.st[node];
      const double* cn = cbuf + (size_t)node * M;
#pragma unroll
      for (int j = 0; j < APT; ++j) c[j] = cn[G::atom(tid, j)];
    }
    uint32_t selm = 0;   // bit j: the thread's atom j is selected
    int t = 0;
    while (st == ST_RUN) {
      // (1) arg-max |c| (lowest index on ties); selected atoms hold exact
      // zeros.
      double bc;
      int bj;
      lane_best(c, bc, bj);
      int bi = G::atom(tid, bj);
      if (bi >= M) bi = M;   // threads without atoms (N <= 8) hold c = 0
      wave_best(bc, bi, bc, bi);
      if (lane == 0) {
        sBc[ph][wv] = bc;
        sBi[ph][wv] = bi;
      }
      __syncthreads();
      bc = sBc[ph][0];
      bi = sBi[ph][0];
#pragma unroll
      for (int q = 1; q < G::NT / 64; ++q) {
        const double oc = sBc[ph][q];
        const int oi = sBi[ph][q];
        if (fabs(oc) > fabs(bc) || (fabs(oc) == fabs(bc) && oi < bi)) {
          bc = oc;
          bi = oi;
        }
      }
      ph ^= 1;
      if (bc == 0.0) {
        st = ST_ZERO;
        break;
      }
      // (2)-(5) in wave 0 (t <= 64 lanes), synchronised within the wave:
      // g_r = <phi_{S_r}, phi_i>; w = L g; d = sqrt(1 - w.w);
      // z_t = <y, q_t> = <r, phi_i> / d (q_t, the new orthonormal direction,
      // is phi_i minus its projection on the selected atoms, over d, and r
      // is orthogonal to those); the new row t of L, (-w^T L, 1) / d;
      // x_S = L^T z updated in place, dx = z_t L[t][:] (x_r += dx_r,
      // x_t = dx_t); the selected atoms listed per family with dx (with x
      // for small blocks) for the refresh.
      if (wv == 0) {
        const int fi = bi / K, pi = bi % N, qi = (bi % K) / N;
        const bool act = lane < t;
        int as = bi;
        double g = 0.0;
        if (act) {
          as = sS[lane];
          if constexpr (NFAM == 2) {
            const int fs = as / K, ps = as % N, qs = (as % K) / N;
            if (fs != fi) g = fi == 0 ? sX[pi][ps] * sX[qi][qs] : sX[ps][pi] * sX[qs][qi];
          }
        }
        sG[lane] = g;
        wave_sync();
        const double* lrow = sLdyn + (lane < k8 ? lane : k8 - 1) * ldl;
        double wr = 0.0;
        for (int c8 = 0; c8 < t; c8 += 8) {
          double lv8[8], g8[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            lv8[i] = lrow[c8 + i];
            g8[i] = sG[c8 + i];
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) wr = fma(lv8[i], g8[i], wr);
        }
        wr = act ? wr : 0.0;
        sW[lane] = wr;
        wave_sync();
        // w L: the first eight rows beside the norm and its root, the others behind
        const double* lcol = sLdyn + (lane < k8 ? lane : k8 - 1);
        auto wl = [&](int r8, double acc) -> double {
          double lv8[8], w8[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            lv8[i] = lcol[(r8 + i) * ldl];
            w8[i] = sW[r8 + i];
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) acc = fma(w8[i], lv8[i], acc);
          return acc;
        };
        double acc = wl(0, 0.0);
        const double s1 = wave_sum_f64(wr * wr);
        const double d2 = 1.0 - s1;
        const bool dep = !(d2 > 1e-24);   // chosen atom (numerically) in the span of the selected ones
        double enew = e;
        if (!dep) {
          const double d = sqrt(d2);
          const double invd = 1.0 / d;
          const double zt = bc / d;
          enew = fma(-zt, zt, e);
          double lr = invd, dx = zt * invd, xn = dx;
          for (int r8 = 8; r8 < t; r8 += 8) acc = wl(r8, acc);
          if (act) {
            lr = -acc * invd;
            dx = zt * lr;
            xn = sXc[lane] + dx;
          }
          const bool in = lane <= t;
          if (lane < k8) sLdyn[t * ldl + lane] = in ? lr : 0.0;
          if (in) sXc[lane] = xn;
          if (lane == 0) {
            sS[t] = bi;
          }
          if constexpr (NFAM == 2) {
            const int f = as / K;
            const unsigned long long m1 = __ballot(in && f == 1), m0 = __ballot(in && f == 0);
            const unsigned long long below = (1ull << lane) - 1ull;
            if (in) {
              const int rk = __popcll((f ? m1 : m0) & below);
              sPQ[f][rk] = (as % N) | (((as % K) / N) << 8);
              sXF[f][rk] = SMALL ? xn : dx;
            }
            const int n0 = __popcll(m0), n1 = __popcll(m1);
            if (lane == 0) {
              sNF[0] = n0;
              sNF[1] = n1;
            }
          }
        }
        if (lane == 0) {
          sScal[0] = dep ? 1.0 : 0.0;
          sScal[1] = enew;
        }
      }
      __syncthreads();
      if (sScal[0] != 0.0) {
        st = ST_ZERO;
        break;
      }
      e = sScal[1];
      if (tid == G::owner(bi)) selm |= 1u << G::slot(bi);
      ++t;
      if (e < eps2)
        st = ST_ACC;
      else if (t >= kmax)
        st = ST_SPARSE;
      if (st != ST_RUN) break;
      // (6) refresh: small blocks c = c0 - G_{:,S} x_S, larger ones
      // c -= G_{:,S} dx (c = c0 - G x at every step either way)
      if constexpr (SMALL) {
#pragma unroll
        for (int f = 0; f < APT; ++f) c[f] = c0[f];
      }
      if constexpr (NFAM == 2 && SMALL) {
        // each of the lane's atoms takes the other family's selections, in
        // selection order, with their current coefficients
        const int qa = tid / N;
        if (tid < K) {
#pragma unroll
          for (int fs = 0; fs < 2; ++fs) {
            const int ns = sNF[fs];
            for (int k0 = 0; k0 < ns; k0 += 4) {   // four at a time: the loads together
              double g[4], x[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int pq = sPQ[fs][k0 + i];
                const int ps = pq & 255, qs = pq >> 8;
                g[i] = fs == 0 ? sX[ps][pa] * sX[qs][qa] : sX[pa][ps] * sX[qa][qs];
                x[i] = sXF[fs][k0 + i];
              }
#pragma unroll
              for (int i = 0; i < 4; ++i) c[1 - fs] = fma(-x[i], g[i], c[1 - fs]);
            }
          }
        }
      } else if constexpr (NFAM == 2 && G::MF) {
        // Each family's atoms take the other family's selections, four at a
        // time as one rank-4 FP64 MFMA update per 16 x 16 tile:
        // C[p][q] += A[p][k] B[k][q] with A = -dx_k X(p part), B = X(q part)
        // (lane: A[lane % 16][lane / 16], B[lane / 16][lane % 16]).
        constexpr int TPW = G::TPW, NT16 = G::NT16;
        const int lk = lane >> 4, li = lane & 15;
#pragma unroll
        for (int fs = 0; fs < 2; ++fs) {
          const int ns = sNF[fs], fa = 1 - fs;   // fa: the family whose atoms change
          for (int kb = 0; kb < ns; kb += 8) {
            // eight selections: two updates whose operands load together
            double xs[2], av[2][TPW], bv[2][TPW];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int pq = sPQ[fs][kb + 4 * u + lk];
              xs[u] = sXF[fs][kb + 4 * u + lk];
              const int ps = pq & 255, qs = pq >> 8;
#pragma unroll
              for (int i = 0; i < TPW; ++i) {
                const int tt = wv * TPW + i, tp = tt / NT16, tq = tt % NT16;
                // family-1 atoms: X[ps][p] X[qs][q]; family-0 atoms: X[p][ps] X[q][qs]
                av[u][i] = fs == 0 ? sX[ps][16 * tp + li] : sX[16 * tp + li][ps];
                bv[u][i] = fs == 0 ? sX[qs][16 * tq + li] : sX[16 * tq + li][qs];
              }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              if (kb + 4 * u >= ns) continue;
#pragma unroll
              for (int i = 0; i < TPW; ++i) {
                const int j0 = fa * G::AF + 4 * i;
                d4 cv = d4{c[j0], c[j0 + 1], c[j0 + 2], c[j0 + 3]};
                cv = mfma64(-xs[u] * av[u][i], bv[u][i], cv);
                c[j0] = cv[0];
                c[j0 + 1] = cv[1];
                c[j0 + 2] = cv[2];
                c[j0 + 3] = cv[3];
              }
            }
          }
        }
      }
#pragma unroll
      for (int j = 0; j < APT; ++j) c[j] = ((selm >> j) & 1u) ? 0.0 : c[j];
    }
    // records: the atoms in selection order with their final coefficients
    if (tid < t) {
      lv.rec_idx[(size_t)node * lv.kmax + tid] = sS[tid];
      lv.rec_coef[(size_t)node * lv.kmax + tid] = sXc[tid];
    }
    if (tid == 0) {
      lv.e[node] = e;
      lv.t[node] = t;
      lv.st[node] = st;
      sNode[np] = (int)gridDim.x + atomicAdd(queue + qk * kQueuePad, 1) * kQueues + qk;
    }
    __syncthreads();   // the next node; sS, sXc are read
  }
}

}  // namespace

hipError_t launch_gram_init(int n, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t lg, int32_t nfam,
                            const double* tab, double* cbuf, hipStream_t s) {
  if (nfam != 1 && nfam != 2) return hipErrorInvalidValue;
#define AQMP_GINIT(NN, GRID)                                                                                  \
  case NN:                                                                                                    \
    if (nfam == 2)                                                                                            \
      hipLaunchKernelGGL((k_gram_init<NN, 2>), dim3(GRID), dim3(256), 0, s, jobs, lv, count, lg, tab, cbuf); \
    else                                                                                                      \
      hipLaunchKernelGGL((k_gram_init<NN, 1>), dim3(GRID), dim3(256), 0, s, jobs, lv, count, lg, tab, cbuf); \
    break;
  switch (n) {
    AQMP_GINIT(16, 2048)
    AQMP_GINIT(32, 1024)
    AQMP_GINIT(64, 512)
    default:
      return hipErrorInvalidValue;
  }
#undef AQMP_GINIT
  return hipGetLastError();
}

hipError_t launch_gram_pursuit(int n, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue, int32_t lg,
                               int32_t nfam, int64_t cap, const double* tab, const double* xg, hipStream_t s) {
  if (nfam == 2 && !xg) return hipErrorInvalidValue;
  if (nfam != 1 && nfam != 2) return hipErrorInvalidValue;
  int dev = 0, n_cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
#define AQMP_GSMALL(KERN, NODES, WGS, ...)   /* fewest nodes per workgroup, workgroups per CU */ \
  {                                                                                       \
    int64_t wgs = (cap + (NODES) - 1) / (NODES);                                          \
    if (wgs > (int64_t)n_cus * (WGS)) wgs = (int64_t)n_cus * (WGS);                       \
    if (wgs < 1) wgs = 1;                                                                 \
    if (nfam == 2)                                                                        \
      hipLaunchKernelGGL((KERN<2>), dim3((unsigned)wgs), dim3(256), 0, s, __VA_ARGS__);   \
    else                                                                                  \
      hipLaunchKernelGGL((KERN<1>), dim3((unsigned)wgs), dim3(256), 0, s, __VA_ARGS__);   \
  }
#define AQMP_GPUR_F(NN, FF)                                                                                 \
  {                                                                                                         \
    int per_cu = 0;                                                                                         \
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_gram_pursuit<NN, FF>, 256, 0) != hipSuccess || \
        per_cu < 1)                                                                                         \
      per_cu = 1;                                                                                           \
    int64_t wgs = (cap + PurGeo<NN, FF>::NPW - 1) / PurGeo<NN, FF>::NPW;                                    \
    if (wgs > (int64_t)n_cus * per_cu) wgs = (int64_t)n_cus * per_cu;                                       \
    if (wgs < 1) wgs = 1;                                                                                   \
    hipLaunchKernelGGL((k_gram_pursuit<NN, FF>), dim3((unsigned)wgs), dim3(256), 0, s, jobs, lv, count, queue, lg, \
                       tab, xg);                                                                            \
  }
#define AQMP_GPUR(NN)    \
  case NN:               \
    if (nfam == 2)       \
      AQMP_GPUR_F(NN, 2) \
    else                 \
      AQMP_GPUR_F(NN, 1) \
    break;
  switch (n) {
    // four waves per SIMD of 16-lane slots, at most a slot per node
    case 4:
      AQMP_GSMALL(k_gram4, 16, 4, jobs, lv, count, tab, xg)
      break;
    case 8:
      AQMP_GSMALL(k_gram8, 4, 4, jobs, lv, count, queue, tab, xg)
      break;
    AQMP_GPUR(16)
    AQMP_GPUR(32)
    AQMP_GPUR(64)
    default:
      return hipErrorInvalidValue;
  }
#undef AQMP_GSMALL
#undef AQMP_GPUR
#undef AQMP_GPUR_F
  return hipGetLastError();
}

hipError_t launch_omp_pursuit(int n, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue, int32_t lg,
                              int32_t nfam, const double* tab, const double* xg, const double* cbuf, int32_t kmax,
                              hipStream_t s) {
  if (nfam == 2 && !xg) return hipErrorInvalidValue;
  if (nfam != 1 && nfam != 2) return hipErrorInvalidValue;
  if (kmax > kOmpMaxAtoms) return hipErrorInvalidValue;
  const int k8 = kmax < 1 ? 8 : (kmax + 7) / 8 * 8;
  int dev = 0, n_cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const size_t smem = sizeof(double) * (size_t)k8 * (k8 + 1);
  // Nodes come from a counter, so the grid is as many workgroups as fit on
  // the device at once (registers and LDS decide; more would only start
  // after the work is gone).
#define AQMP_OMP_F(NN, FF)                                                                                     \
  {                                                                                                            \
    int per_cu = 0;                                                                                            \
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_omp<NN, FF>, OmpGeo<NN, FF>::NT, smem) !=     \
            hipSuccess ||                                                                                      \
        per_cu < 1)                                                                                            \
      per_cu = 1;                                                                                              \
    hipLaunchKernelGGL((k_omp<NN, FF>), dim3(n_cus * per_cu), dim3(OmpGeo<NN, FF>::NT), smem, s, jobs, lv,  \
                       count, queue, lg, tab, xg, cbuf, k8);                                                  \
  }
#define AQMP_OMP(NN)             \
  case NN:                       \
    if (nfam == 2)               \
      AQMP_OMP_F(NN, 2)          \
    else                         \
      AQMP_OMP_F(NN, 1)          \
    break;
  switch (n) {
    AQMP_OMP(4)
    AQMP_OMP(8)
    AQMP_OMP(16)
    AQMP_OMP(32)
    AQMP_OMP(64)
    default:
      return hipErrorInvalidValue;
  }
#undef AQMP_OMP
#undef AQMP_OMP_F
  return hipGetLastError();
}

}  // namespace aqmp
