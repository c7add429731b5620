// kernels_tree.hip - the quadtree worklist on the device: stable stream
// compaction of the active nodes and split/child emission (Algorithm 2).
// All of it is integer work with a fixed result: a single-pass prefix sum
// with decoupled look-back keeps the original order of the kept items.
#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

// Completion count of a look-back scan by `blocks` blocks; the last one to
// finish clears the tile words and the tickets for the next launch.
__device__ void scan_done(ScanState ss, int ntiles, int blocks) {
  __shared__ int s_last;
  const int tid = threadIdx.x;
  __syncthreads();
  if (tid == 0) {
    __threadfence();
    const int done = atomicAdd(&ss.ticket[1], 1);
    s_last = (done == blocks - 1);
  }
  __syncthreads();
  if (s_last) {
    for (int i = tid; i < ntiles && i < ss.ntiles_max; i += blockDim.x) ss.tiles[i] = 0ull;
    if (tid == 0) {
      ss.ticket[0] = 0;
      ss.ticket[1] = 0;
    }
  }
}

// One launch = one stable scan over op.count() items with 0/1 keep flags.
// Blocks take tiles in ticket order, so a block only ever waits on tiles
// owned by blocks that started before it.  Every wait is bounded; when a
// bound runs out the scan reports it through *err and continues (its output
// is then wrong, and the host turns the flag into an error).  The last block
// to finish clears the tile words and the tickets for the next launch.
template <class Op>
__device__ void stable_scan(Op& op, ScanState ss, int32_t* err) {
  __shared__ int s_tile, s_prefix;
  __shared__ int s_wsum[4];
  const int tid = threadIdx.x;
  if (tid == 0) s_tile = atomicAdd(&ss.ticket[0], 1);
  __syncthreads();
  const int tile = s_tile;
  const int n = op.count();
  const int ntiles = (n + kScanTile - 1) / kScanTile;
  if (tile < ntiles) {
    const int base = tile * kScanTile + tid * 4;
    int f[4];
    int loc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = base + j;
      f[j] = (i < n) ? op.keep(i) : 0;
      loc += f[j];
    }
    const int lane = tid & 63, w = tid >> 6;
    int x = loc;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) s_wsum[w] = x;
    __syncthreads();
    int wpre = 0;
    for (int j = 0; j < w; ++j) wpre += s_wsum[j];
    const int agg = s_wsum[0] + s_wsum[1] + s_wsum[2] + s_wsum[3];
    const int excl = wpre + x - loc;
    if (w == 0) {
      const int pre = lookback_wave(ss.tiles, tile, agg, err);
      if (lane == 0) s_prefix = pre;
    }
    __syncthreads();
    int pos = s_prefix + excl;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (f[j]) op.emit(base + j, pos++);
    }
    if (tile == ntiles - 1 && tid == 0) op.total(s_prefix + agg);
  } else if (tile == 0 && tid == 0) {
    op.total(0);   // n == 0: nothing kept
  }
  scan_done(ss, ntiles, (int)gridDim.x);
}

struct CompactOp {
  const int32_t* in_list;   // null = identity (item i is node i)
  const int32_t* in_count;
  const uint8_t* st;
  int32_t* out_list;
  int32_t* out_count;
  int32_t* clear;           // optional counter set to zero with the total
  __device__ int count() const { return *in_count; }
  __device__ int node(int i) const { return in_list ? in_list[i] : i; }
  __device__ int keep(int i) const { return st[node(i)] == ST_RUN ? 1 : 0; }
  __device__ void emit(int i, int pos) const { out_list[pos] = node(i); }
  __device__ void total(int t) const {
    *out_count = t;
    if (clear) *clear = 0;
  }
};

__global__ __launch_bounds__(256) void k_compact(CompactOp op, ScanState ss, int32_t* err) {
  stable_scan(op, ss, err);
}

struct SplitOp {
  const JobDev* jobs;
  int32_t n_jobs;
  int32_t* bad;             // set when a node names a job outside the table
  LevelDev parent;
  const int32_t* parent_count;
  LevelDev child;
  int32_t child_ntop;
  int32_t* child_count;
  int2* child_ranges;       // per job, or null
  int32_t lg;
  // Algorithm 2: refine when N > N_min and the node failed the test of its
  // split rule; the node's own atoms are then discarded by the exporter.
  __device__ bool split(int jb, double e, int t) const {
    if ((unsigned)jb >= (unsigned)n_jobs) return false;
    const JobDev& j = jobs[jb];
    const int n_min = j.n_min, rule = j.split_rule, k = j.k[lg];
    const double eps2 = j.eps2[lg];
    return (1 << lg) > n_min && (rule == AQMP_SPLIT_R1 ? e >= eps2 : t >= k);
  }
};

// The split test of a level's nodes and its children, in the nodes' order:
// child 4 p + q is quadrant q (TL, TR, BL, BR) of the p-th split node.  One
// node per thread, 1024 per workgroup (tile).
// What bounds it: the chain of loads (each from the far cache, since other
// XCDs wrote the nodes) and the look-back from tile to tile.  So a node's
// values are all loaded before any is used, a tile that is alone takes no
// ticket, and the workgroups past the level's last tile (the grid covers its
// capacity) leave before the tickets.  Mean of a launch, with four nodes per
// thread, one value at a time, and tickets for every workgroup before: one
// tile 7.1 -> 4.4 us; 3072, 5136 and 12 892 nodes 12.9 -> 7.6 us; 6144 to
// 64 352 nodes 19.8 -> 8.7 us.  (Splits of earlier tiles counted by reading
// their nodes again, no look-back: 7.3 us for the middle ones, 9.0 for the
// last.)
__global__ __launch_bounds__(kScanTile) void k_split_emit(SplitOp op, ScanState ss, int32_t* err) {
  constexpr int NW = kScanTile / 64;
  __shared__ int s_tile, s_prefix;
  __shared__ int s_own[NW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = *op.parent_count;
  const int ntiles = (n + kScanTile - 1) / kScanTile;
  int tile = (int)blockIdx.x;
  if (tile >= ntiles) {   // the grid covers the level's capacity
    if (tile == 0 && tid == 0) *op.child_count = op.child_ntop;
    return;
  }
  if (ntiles > 1) {   // the ntiles blocks that are left share the tickets
    if (tid == 0) s_tile = atomicAdd(&ss.ticket[0], 1);
    __syncthreads();
    tile = s_tile;
  }
  const int i = tile * kScanTile + tid;
  const bool in = i < n;
  int jb = -1, jprev = -1, jnext = -1, x = 0, y = 0, t = 0;
  double e = 0.0;
  uint8_t st = 0;
  if (in) {
    jb = op.parent.job[i];
    e = op.parent.e[i];
    t = op.parent.t[i];
    x = op.parent.x0[i];
    y = op.parent.y0[i];
    st = op.parent.st[i];
    if (op.child_ranges) {
      if (i > 0) jprev = op.parent.job[i - 1];
      if (i < n - 1) jnext = op.parent.job[i + 1];
    }
  }
  const bool keep = in && op.split(jb, e, t);
  if (in && (unsigned)jb >= (unsigned)op.n_jobs) atomicExch(op.bad, 1);
  if (keep) op.parent.st[i] = (uint8_t)(st | ST_SPLIT);
  const unsigned long long mask = __ballot(keep);
  if (lane == 0) s_own[wv] = __popcll(mask);
  __syncthreads();
  int pre = 0, agg = 0, pos = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    pos += w < wv ? s_own[w] : 0;
    agg += s_own[w];
  }
  if (ntiles > 1) {
    if (wv == 0) {
      const int p = lookback_wave(ss.tiles, tile, agg, err);
      if (lane == 0) s_prefix = p;
    }
    __syncthreads();
    pre = s_prefix;
  }
  pos += pre + __popcll(mask & ((1ull << lane) - 1ull));
  if (in && op.child_ranges && (unsigned)jb < (unsigned)op.n_jobs) {
    // The nodes of a job are neighbours: top-level nodes are listed job by
    // job and children come in their parents' order, so its first and last
    // node, with the splits before them, give its children's range.
    if (i == 0 || jprev != jb) op.child_ranges[jb].x = op.child_ntop + 4 * pos;
    if (i == n - 1 || jnext != jb) op.child_ranges[jb].y = op.child_ntop + 4 * (pos + (keep ? 1 : 0));
  }
  if (keep) {
    const int h = 1 << (op.lg - 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = op.child_ntop + 4 * pos + q;
      op.child.job[c] = jb;
      op.child.x0[c] = x + (q & 1) * h;
      op.child.y0[c] = y + (q >> 1) * h;
    }
  }
  if (tile == ntiles - 1 && tid == 0) *op.child_count = op.child_ntop + 4 * (pre + agg);
  if (ntiles > 1) scan_done(ss, ntiles, ntiles);
}

// Word 0 = v, words 1 .. n-1 = 0: one thread per word.
__global__ __launch_bounds__(256) void k_head_zero_u32(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = i == 0 ? v : 0u;
}

static_assert(kLevels * kQueues <= 64, "one thread per counter");
static_assert(sizeof(ExportTotals) <= 64 * 8, "one thread per total");
__global__ void k_init_counts(Counters* c, Queues* q, ExportTotals* tot, const int32_t* ntop) {
  const int i = threadIdx.x;
  if (i < kLevels) c->count[i] = ntop[i];
  if (i < 3) c->act[i] = 0;
  if (i == 0) c->scan_error = 0;
  if (i < (int)(sizeof(ExportTotals) / 8)) ((unsigned long long*)tot)[i] = 0ull;
  if (i < kLevels * kQueues) q->at[i / kQueues][(i % kQueues) * kQueuePad] = 0;
}

}  // namespace

hipError_t launch_init_counts(Counters* c, Queues* q, ExportTotals* tot, const int32_t* ntop_dev, hipStream_t s) {
  hipLaunchKernelGGL(k_init_counts, dim3(1), dim3(64), 0, s, c, q, tot, ntop_dev);
  return hipGetLastError();
}

hipError_t launch_head_zero_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t b = (n + 255) / 256;
  if (b > 1024) b = 1024;
  hipLaunchKernelGGL(k_head_zero_u32, dim3((unsigned)b), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

static int scan_blocks(int64_t cap) {
  int64_t b = (cap + kScanTile - 1) / kScanTile;
  return (int)(b < 1 ? 1 : b);
}

hipError_t launch_compact(const int32_t* in_list, const int32_t* in_count, const uint8_t* st,
                          int32_t* out_list, int32_t* out_count, int32_t* clear_count, int64_t cap,
                          ScanState ss, int32_t* err, hipStream_t s) {
  CompactOp op{in_list, in_count, st, out_list, out_count, clear_count};
  hipLaunchKernelGGL(k_compact, dim3(scan_blocks(cap)), dim3(256), 0, s, op, ss, err);
  return hipGetLastError();
}

hipError_t launch_split_emit(const JobDev* jobs, int32_t n_jobs, LevelDev parent, const int32_t* parent_count,
                             LevelDev child, int32_t child_ntop, int32_t* child_count, int2* child_ranges,
                             int32_t lg, int64_t cap, ScanState ss, int32_t* err, hipStream_t s) {
  SplitOp op{jobs, n_jobs, err, parent, parent_count, child, child_ntop, child_count, child_ranges, lg};
  hipLaunchKernelGGL(k_split_emit, dim3(scan_blocks(cap)), dim3(kScanTile), 0, s, op, ss, err);
  return hipGetLastError();
}

}  // namespace aqmp
