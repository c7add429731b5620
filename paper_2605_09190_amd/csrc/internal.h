// internal.h - structures shared by the host orchestration and the kernels
// of the AQMP encoder library.  Not part of the public ABI (see aqmp.h).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <mutex>
#include <utility>
#include <vector>

#include "aqmp.h"

namespace aqmp {

// Node status byte.  The low two bits say why MP stopped (or that it is still
// running); ST_SPLIT is set by the split pass.
enum : uint8_t {
  ST_RUN = 0,       // MP continues at the next step
  ST_ACC = 1,       // stopped: ||r||^2 < eps_N^2 (eq. (2), accuracy)
  ST_SPARSE = 2,    // stopped: k_N iterations made (eq. (2), sparsity)
  ST_ZERO = 3,      // stopped: the largest |correlation| is exactly zero
  ST_SPLIT = 0x10,  // node refined into its four quadrants
};

constexpr int kLevels = 7;        // log2(N) for N = 1 .. 64
constexpr int kCand = AQMP_CANDIDATES;
constexpr int kTopR = 8;          // keys kept per node per atom tile
constexpr int kScanTile = 1024;   // items per block of the stable scans
constexpr int kFusedMaxN = 8;     // levels up to this size run as one launch in every form
constexpr int kBranches = 4;      // parallel graph branches of the concurrent schedule
constexpr int kOmpMaxAtoms = AQMP_OMP_MAX_ATOMS;   // OMP: selected atoms per node (LDS factor size)
constexpr int kQueues = 8, kQueuePad = 32;   // node queues of a level and the words between them
constexpr int kSsimMomentBlocks = 1024;   // workgroups of the whole-plane SSIM moments

// Kernel launch, with start/end events recorded by the dispatch when given.
template <typename F, typename... Args>
inline void launch_timed(F kernel, dim3 grid, dim3 block, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                         Args... args) {
  if (ev0 || ev1)
    hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev0, ev1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
}

inline int ilog2(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// Per-job table read by the kernels.  eps2 and k are indexed by log2(N).
struct JobDev {
  const void* img;
  int32_t dtype;
  int32_t w, h;
  int32_t n_min, n_max;
  int32_t split_rule;
  int64_t row_stride;
  double eps2[kLevels];
  int32_t k[kLevels];
  int32_t pad;
};

// Planes are device memory: global loads (a pointer taken from the job table
// is generic to the compiler, and a flat load also waits on the LDS counter).
typedef __attribute__((address_space(1))) double gmem_f64;
typedef __attribute__((address_space(1))) float gmem_f32;

// Pixel (y, x) of a job's plane in FP64.  Blocks tile the plane padded up
// to a multiple of N_max; rows and columns past the image repeat its last
// row and column (edge replication).
__device__ inline double job_pixel(const JobDev& jb, int y, int x) {
  y = y < jb.h ? y : jb.h - 1;
  x = x < jb.w ? x : jb.w - 1;
  const int64_t idx = (int64_t)y * jb.row_stride + x;
  return jb.dtype == AQMP_F64 ? ((const gmem_f64*)jb.img)[idx] : (double)((const gmem_f32*)jb.img)[idx];
}

// Host checks of one parameter set (AQMP_E_INVALID with tag + reason), and
// the per-job table entry the kernels read for a plane and a parameter set.
int check_params(const aqmp_params& p, const std::string& tag);
JobDev make_jobdev(const aqmp_image& im, const aqmp_params& p);

// Pixels (y, x0 .. x0 + W - 1) of a job's plane in FP64, edge-replicated
// like job_pixel.  The sample type is tested once and the W loads are
// independent, so they are all in flight together.
template <int W>
__device__ inline void job_pixels(const JobDev& jb, int y, int x0, double (&v)[W]) {
  const int yy = y < jb.h ? y : jb.h - 1;
  const int64_t row = (int64_t)yy * jb.row_stride;
  int xs[W];
#pragma unroll
  for (int j = 0; j < W; ++j) xs[j] = x0 + j < jb.w ? x0 + j : jb.w - 1;
  if (jb.dtype == AQMP_F64) {
    const gmem_f64* p = (const gmem_f64*)jb.img + row;
#pragma unroll
    for (int j = 0; j < W; ++j) v[j] = p[xs[j]];
  } else {
    const gmem_f32* p = (const gmem_f32*)jb.img + row;
#pragma unroll
    for (int j = 0; j < W; ++j) v[j] = (double)p[xs[j]];
  }
}

// Device-side arrays of one quadtree level (block size N = 1 << lg).  The
// node arrays are shared by all passes; a pass owns [base, base + cap).
struct LevelDev {
  int32_t* job;
  int32_t* x0;
  int32_t* y0;
  double* e;        // ||r||^2 after the last iteration (FP64)
  int32_t* t;       // iterations made
  uint8_t* st;      // ST_* status
  int32_t* rec_idx;   // [node * kmax + t] selected atom
  double* rec_coef;   // [node * kmax + t] FP64 coefficient
  int32_t kmax;
};

// Per-pass counters in device memory.
struct Counters {
  int32_t count[kLevels];   // nodes present at each level
  int32_t act[3];           // active-list lengths (rotating: in, out, cleared)
  int32_t scan_error;       // set if a bounded scan wait ran out
  int32_t pad;
};

// Work counters of the pursuits whose nodes are taken by many small workers:
// kQueues per level, a cache line each, queue q handing out every kQueues-th
// node.  (Thousands of workers on one counter waited in line for it: about
// 12 ns each, 25 us for 2 048 waves that start together.)
struct Queues {
  int32_t at[kLevels][kQueues * kQueuePad];
};
// The next node of a worker that takes from queue qk, the first q0 nodes
// having been dealt out; when its queue is empty, one of another that is not
// (qk then names that one).  `count` or more: none is left.
__device__ inline int next_node(int32_t* queue, int& qk, int q0, int count) {
  int node = q0 + atomicAdd(queue + qk * kQueuePad, 1) * kQueues + qk;
  if (node < count) return node;
  int at[kQueues];
#pragma unroll
  for (int k = 1; k < kQueues; ++k)
    at[k] = __hip_atomic_load(queue + (qk + k) % kQueues * kQueuePad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int own = qk;
#pragma unroll
  for (int k = 1; k < kQueues; ++k) {
    const int q = (own + k) % kQueues;
    if (node >= count && q0 + at[k] * kQueues + q < count) {
      node = q0 + atomicAdd(queue + q * kQueuePad, 1) * kQueues + q;
      qk = q;
    }
  }
  return node;
}

// Look-back scan bookkeeping: one 64-bit word per tile plus two counters.
// The last block of every scan launch restores it to zero.
struct ScanState {
  unsigned long long* tiles;
  int32_t* ticket;   // [0] tile ticket, [1] blocks done
  int32_t ntiles_max;
};

// Arguments of the per-step kernels of one level.
struct StepArgs {
  const JobDev* jobs;
  LevelDev lv;            // already offset by the pass base
  int32_t lg;             // log2(N)
  int32_t n_atoms;        // M (real atoms; the correlation pads to its tile)
  int32_t nfam;
  const double* tab;      // FP64 1D tables [nfam][N][N]
  const float* tabT32;    // the same rounded to FP32 and transposed, [nfam][pixel][row]
  float* r32;             // residual [node][N*N] FP32, row-major pixels
  uint16_t* r16;          // BF16 shadow of r32 (null in the FP32 form)
  const int32_t* act;     // active list (node slots within the pass)
  const int32_t* act_count;
  unsigned long long* keys;   // [pos][atom tile][kTopR]
  int32_t n_atom_tiles;
  // The select step appends the nodes still running to next_act (any
  // order; zero on entry) and zeroes clear_count, the counter the step
  // after the next one appends to.  next_act is null on a level's last step.
  int32_t* next_act;
  int32_t* next_count;
  int32_t* clear_count;
  // Node-tile range of the generated-atom correlation: lo | hi << 4, 0 =
  // the kernel's own range.
  int32_t corr_tile;
};

// ---------------------------------------------------------------------------
// Launch wrappers (defined in the kernel translation units).
// ---------------------------------------------------------------------------
struct ExportTotals;
// Sets a pass's counters and queues, and clears the code's totals.
hipError_t launch_init_counts(Counters* c, Queues* q, ExportTotals* tot, const int32_t* ntop_dev, hipStream_t s);
// p[0] = v and p[1 .. n-1] = 0, by a fill kernel.
hipError_t launch_head_zero_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s);
hipError_t launch_gather(int n, const StepArgs& a, const int32_t* count, hipStream_t s);
hipError_t launch_compact(const int32_t* in_list, const int32_t* in_count, const uint8_t* st,
                          int32_t* out_list, int32_t* out_count, int32_t* clear_count, int64_t cap,
                          ScanState ss, int32_t* err, hipStream_t s);
// Split test and child emission of one level.  A node whose job index is not
// below n_jobs is not split and sets *err.  child_ranges, when given, receives
// per job of the level the range of its children (their jobs keep their order).
hipError_t launch_split_emit(const JobDev* jobs, int32_t n_jobs, LevelDev parent, const int32_t* parent_count,
                             LevelDev child, int32_t child_ntop, int32_t* child_count, int2* child_ranges,
                             int32_t lg, int64_t cap, ScanState ss, int32_t* err, hipStream_t s);
// ev0 / ev1, when given, are recorded by the dispatch itself at the kernel's
// start and end (hipExtLaunchKernel), so their elapsed time is the kernel's
// execution time without the launch gap.
hipError_t launch_corr(int n, int precision, int variant, const void* dict_atoms, const StepArgs& a,
                       int32_t m_pad, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t launch_select(int n, const StepArgs& a, int64_t cap, hipStream_t s, hipEvent_t ev0 = nullptr,
                         hipEvent_t ev1 = nullptr);
// Whole-level pursuit of the dense solver at N = 32 and 64 with the
// correlation factored through the atoms' outer products (`queue`: the level's
// node counters, zero on entry; cap: its node capacity; ops: the table
// operands launch_sep_ops made, sep_ops_bytes long, 0 for other N).
size_t sep_ops_bytes(int n, uint32_t families);
hipError_t launch_sep_ops(int n, uint32_t families, const double* tab, const double* xg, void* out, hipStream_t s);
hipError_t launch_pursuit_sep(int n, uint32_t families, const JobDev* jobs, LevelDev lv, const int32_t* count,
                              int32_t* queue, int64_t cap, const double* tab, const void* ops, hipStream_t s);
hipError_t launch_mp_fused4(const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t lg, int32_t n_atoms,
                            const double* tab, hipStream_t s);
// Whole-level pursuit of the dense solver at N = 8 and 16
// (queue: the level's node counters, zero on entry; cap: its node capacity).
hipError_t launch_pursuit_sub(int n, int precision, uint32_t families, const JobDev* jobs, LevelDev lv,
                              const int32_t* count, int32_t* queue, int64_t cap, const double* tab, const double* xg,
                              hipStream_t s);
// Gram and OMP forms (FP64).  launch_gram_pursuit takes each node of the level
// through its whole MP (Gram updates).  launch_omp_pursuit does so for OMP
// (least-squares refits) with, for N >= 16, the initial correlations that
// launch_gram_init wrote to cbuf ([node][nfam * n * n]) before it, together
// with each node's ||y||^2 and first stop test.  `queue`: the level's node
// counters, zero on entry; cap: its node capacity.
hipError_t launch_gram_init(int n, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t lg, int32_t nfam,
                            const double* tab, double* cbuf, hipStream_t s);
hipError_t launch_gram_pursuit(int n, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue, int32_t lg,
                               int32_t nfam, int64_t cap, const double* tab, const double* xg, hipStream_t s);
// kmax: the largest k among the level's jobs (at most kOmpMaxAtoms); it
// sizes the factor in LDS.
hipError_t launch_omp_pursuit(int n, const JobDev* jobs, LevelDev lv, const int32_t* count, int32_t* queue, int32_t lg,
                              int32_t nfam, const double* tab, const double* xg, const double* cbuf, int32_t kmax,
                              hipStream_t s);
// SSIM partials: one FP64 per workgroup (window7) or five plane sums per
// workgroup (global); *n_partial receives the workgroup count.
hipError_t launch_ssim(const aqmp_image& x, const aqmp_image& y, int mode, double c1, double c2, double* partial,
                       int* n_partial, hipStream_t s);
int ssim_planes(const aqmp_image* x, const aqmp_image* y, int mode, double data_range, double* out, hipStream_t s);
// Decode of one job: its levels (lg_hi .. lg_lo), their FP64 tables, and the
// ranges of every job's nodes per level ([level][job]: first, end).
struct DecodeLevel {
  LevelDev lv;
  const double* tab;
};
struct DecodeArgs {
  DecodeLevel lv[kLevels];
  const JobDev* jobs;
  const int2* ranges;
  int32_t n_jobs, job, lg_hi, lg_lo;
};
// step > 0: every coefficient is replaced by its quantised value
// rint(c / step) * step first (the stream's coefficient format 1).
// blocks_px: pixels of the job's padded plane.
hipError_t launch_decode(const DecodeArgs& a, int64_t blocks_px, double step, void* out, int32_t dtype, int64_t row_stride,
                         hipStream_t s);

// Device gather of a code's visited nodes in canonical order.  Sort key of a
// node: global top-level block ordinal << kExportLowBits | Morton code of its
// corner inside that block << 3 | (7 - log2 N).
constexpr int kExportCornerBits = 6;                       // corner coordinates < 64
constexpr int kExportLowBits = 2 * kExportCornerBits + 3;
struct ExportSeg {          // one level of one pass
  LevelDev L;               // offset by the pass base
  const int32_t* count;     // nodes present (device)
  int32_t lg;
  int32_t cap;              // its node slots
  uint32_t flat_base;       // first flat node id of the segment
};
// What a code holds, by block size, and the slot counter of the key pass.
struct ExportTotals {
  unsigned long long nodes[kLevels], leaves[kLevels], iters[kLevels], emitted[kLevels];
  unsigned long long next;
};
struct ExportJob {
  long long top_base;       // global ordinal of the job's first top-level block
  int32_t nm;               // N_max of the job
  int32_t cols;             // top-level blocks per row of the padded plane
};
hipError_t launch_export_stats(const ExportSeg* segs, int nseg, int64_t max_cap, ExportTotals* tot, hipStream_t s);
hipError_t launch_export_keys(const ExportSeg* segs, int nseg, int64_t max_cap, const ExportJob* jx, bool leaves_only,
                              unsigned long long* keys, uint32_t* vals, unsigned long long* next, hipStream_t s);
hipError_t export_sort(void* tmp, size_t& tmp_bytes, unsigned long long* keys, unsigned long long* keys_out,
                       uint32_t* vals, uint32_t* vals_out, int64_t n, int end_bit, hipStream_t s);
hipError_t export_scan(void* tmp, size_t& tmp_bytes, const int64_t* in, int64_t* out, int64_t n, hipStream_t s);
hipError_t launch_export_counts(const ExportSeg* segs, int nseg, const uint32_t* vals, int64_t n, int64_t* t_out,
                                hipStream_t s);
// The keys, the sort, the counts and the scan in one launch, for n <= kOrderMax
// of at most kOrderVisited nodes in at most kOrderSegs segments.
constexpr int kOrderBits = 11, kOrderMax = 1 << kOrderBits, kOrderVisited = 4096, kOrderSegs = 64;
static_assert(kExportLowBits + 12 + kOrderBits <= 64, "a key of up to 4096 top-level blocks and a place");
hipError_t launch_export_order(const ExportSeg* segs, int nseg, const ExportJob* jx, bool leaves_only, int64_t visited,
                               int64_t n, uint32_t* vals, int64_t* off, hipStream_t s);
hipError_t launch_export_write(const ExportSeg* segs, int nseg, const uint32_t* vals, const int64_t* off, int64_t n,
                               aqmp_leaf* out, int32_t* idx, double* coef, hipStream_t s);

// Name of the correlation kernel launch_corr runs (or the whole-level pursuit
// for n <= kFusedMaxN); "" when the combination is invalid.
const char* corr_kernel_name(int n, int precision, int variant);
// The BF16 correlation variants the library has: 0 (default), 2, 3, 6.
inline bool corr_variant_valid(int v) { return v == 0 || v == 2 || v == 3 || v == 6; }

// Tile geometry of the correlation kernel per block size (atoms per tile).
int corr_atom_tile(int n);
int corr_grid(int n, int precision);

}  // namespace aqmp

// Opaque public handles.
struct aqmp_dict {
  // Streams that capture the graphs of the dictionary's codes: making one takes
  // 460 us, ten times the rest of a capture.  At most kBranches + 1 idle ones
  // are kept (with their device), and given back with the dictionary.
  struct CaptureStreams {
    std::mutex mu;
    std::vector<std::pair<int, hipStream_t>> idle;
  };
  mutable CaptureStreams capture;
  int n_min, n_max;
  uint32_t families;
  int nfam;
  struct Level {
    bool have = false;
    int n = 0, k = 0, m = 0, m_pad = 0;
    std::vector<double> h_tab;     // [nfam][n][n]
    double* d_tab = nullptr;
    float* d_tabT32 = nullptr;     // [nfam][y][p] = fl32(T_f[p][y])
    double* d_xg = nullptr;        // [n][n] <T_0[p], T_1[p']> (two families only)
    float* d_f32 = nullptr;        // [m_pad][k]
    uint16_t* d_bf16 = nullptr;    // [m_pad][k]
    void* d_sep = nullptr;         // operands of the factored correlation (launch_sep_ops)
  } lv[aqmp::kLevels];
};
