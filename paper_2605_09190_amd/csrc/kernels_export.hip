// kernels_export.hip - a code's visited nodes gathered on the device in the
// canonical order of its readers (export, statistics, bitstream): job, then
// top-level block in raster order, then depth-first with the children of a
// node in TL, TR, BL, BR order (Alg. 2 recursion).  Depth-first order inside
// a top-level block is the order of (Morton code of the node's corner,
// larger node first), so one radix sort of a 64-bit key per node gives it.
// The host then reads three dense arrays (node records, atom indices,
// coefficients) instead of every level's fixed-stride record slots; of the
// leaves alone where the caller asks for those (their atoms are about two
// thirds of all).
#include <algorithm>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "internal.h"
#include "dev_common.h"

namespace aqmp {

namespace {

// Morton code of a corner inside its top-level block: x in the even bits,
// so TL < TR < BL < BR at every level.
__device__ inline uint32_t corner_morton(uint32_t x, uint32_t y) {
  uint32_t m = 0;
#pragma unroll
  for (int b = 0; b < kExportCornerBits; ++b) m |= (((x >> b) & 1u) << (2 * b)) | (((y >> b) & 1u) << (2 * b + 1));
  return m;
}

// A node's place in the canonical order.
__device__ inline unsigned long long export_key(const ExportJob& j, int x0, int y0, int lg) {
  const long long top = j.top_base + (long long)(y0 / j.nm) * j.cols + x0 / j.nm;
  return ((unsigned long long)top << kExportLowBits) |
         ((unsigned long long)corner_morton((uint32_t)(x0 % j.nm), (uint32_t)(y0 % j.nm)) << 3) |
         (unsigned long long)(7 - lg);
}

// Flat node id -> its segment (level of a pass), by binary search over the
// segments' first flat ids.
__device__ inline int seg_of(const ExportSeg* segs, int nseg, uint32_t fid) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (segs[mid].flat_base <= fid) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Nodes, leaves, their MP iterations and those of the leaves, per block size:
// a sum per workgroup, then one atomic each.
__global__ __launch_bounds__(256) void k_export_stats(const ExportSeg* segs, ExportTotals* tot) {
  const ExportSeg sg = segs[blockIdx.y];
  const int count = min(*sg.count, sg.cap);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  unsigned long long v[3] = {0, 0, 0};                   // leaves, iterations, iterations of leaves
  for (int i = blockIdx.x * 256 + (int)threadIdx.x; i < count; i += gridDim.x * 256) {
    const int t = sg.L.t[i];
    const bool leaf = !(sg.L.st[i] & ST_SPLIT);
    v[0] += leaf ? 1 : 0;
    v[1] += t;
    v[2] += leaf ? t : 0;
  }
  __shared__ unsigned long long part[4][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v[k] += __shfl_xor(v[k], d, 64);
    if (lane == 0) part[w][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < 3 && (int)blockIdx.x * 256 < count) {
    const int k = threadIdx.x;
    const unsigned long long sum = part[0][k] + part[1][k] + part[2][k] + part[3][k];
    atomicAdd(k == 0 ? &tot->leaves[sg.lg] : (k == 1 ? &tot->iters[sg.lg] : &tot->emitted[sg.lg]), sum);
  }
  if (blockIdx.x == 0 && threadIdx.x == 64) atomicAdd(&tot->nodes[sg.lg], (unsigned long long)count);
}

// One key and one flat id per visited node (or leaf), appended in any order
// (the sort fixes the order); *next is zero on entry.
__global__ __launch_bounds__(256) void k_export_keys(const ExportSeg* segs, const ExportJob* jx, int leaves_only,
                                                     unsigned long long* keys, uint32_t* vals,
                                                     unsigned long long* next) {
  const ExportSeg sg = segs[blockIdx.y];
  const int count = min(*sg.count, sg.cap);
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int base = blockIdx.x * 256; base < count; base += gridDim.x * 256) {
    const int i = base + (int)threadIdx.x;
    const bool v = i < count && !(leaves_only && (sg.L.st[i] & ST_SPLIT));
    unsigned long long key = 0;
    if (v) {
      const int job = sg.L.job[i];
      const ExportJob j = jx[job];
      const int x0 = sg.L.x0[i], y0 = sg.L.y0[i];
      key = export_key(j, x0, y0, sg.lg);
    }
    const unsigned long long m = __ballot(v);
    const int rank = __popcll(m & below);
    unsigned long long slot = 0;
    if (lane == 0 && m) slot = atomicAdd(next, (unsigned long long)__popcll(m));
    slot = __shfl(slot, 0, 64);
    if (v) {
      keys[slot + rank] = key;
      vals[slot + rank] = sg.flat_base + (uint32_t)i;
    }
  }
}

// Atom counts in sorted order (the scan's input).
__global__ __launch_bounds__(256) void k_export_counts(const ExportSeg* segs, int nseg, const uint32_t* vals,
                                                       int64_t n, int64_t* t_out) {
  for (int64_t p = blockIdx.x * 256ll + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
    const uint32_t fid = vals[p];
    const ExportSeg& sg = segs[seg_of(segs, nseg, fid)];
    t_out[p] = sg.L.t[fid - sg.flat_base];
  }
}

// Keys, order and atom offsets of up to kOrderMax nodes in one workgroup: the
// levels' counts, a key per node, a bitonic sort and a prefix sum, all in LDS.
// vals gets the flat ids in order, off the nodes' first atoms.  `size` is a
// power of two, n <= size, two places per thread; the levels hold at most
// kOrderSegs segments and `visited` nodes, so the ordinals of their top-level
// blocks are small and a key leaves room for a place.
// What bounds it: three dependent loads, then the LDS traffic of the sort (28
// passes over 128 places, 66 over 2048; with the places in an array of their
// own a third more, 26 us instead of 21).  64 of 84 nodes 8.6 us, 847 of 1 108
// 21 us; keys, radix sort, counts and scan as launches of their own 15 and 26
// us, and five more launches.
__global__ __launch_bounds__(1024) void k_export_order(const ExportSeg* segs, int nseg, const ExportJob* jx,
                                                       int leaves_only, int visited, int n, int size, uint32_t* vals,
                                                       int64_t* off) {
  __shared__ unsigned long long key[kOrderMax];   // the node's key, then its place in fid and cnt
  __shared__ uint32_t fid[kOrderMax];
  __shared__ int cnt[kOrderMax];
  __shared__ int first[kOrderSegs];
  __shared__ int s_next, s_wave[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nt = blockDim.x;
  if (tid == 0) s_next = 0;
  if (wv == 0) {   // the segments' first nodes
    const int c = lane < nseg ? min(*segs[lane].count, segs[lane].cap) : 0;
    int x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    first[lane] = lane < nseg ? x - c : 0x7fffffff;
  }
  for (int i = tid; i < size; i += nt) key[i] = ~0ull;
  __syncthreads();
  for (int base = 0; base < visited; base += nt) {
    const int v = base + tid;
    int g = 0;
    while (g + 1 < nseg && first[g + 1] <= v) ++g;
    const ExportSeg& sg = segs[g];
    const int i = v - first[g];
    bool keep = v < visited && i < min(*sg.count, sg.cap);
    int t = 0, job = 0, x0 = 0, y0 = 0;
    if (keep) {
      const uint8_t st = sg.L.st[i];
      t = sg.L.t[i];
      job = sg.L.job[i];
      x0 = sg.L.x0[i];
      y0 = sg.L.y0[i];
      keep = !(leaves_only && (st & ST_SPLIT));
    }
    const unsigned long long m = __ballot(keep);
    int slot = 0;
    if (lane == 0 && m) slot = atomicAdd(&s_next, __popcll(m));
    slot = __shfl(slot, 0, 64) + __popcll(m & ((1ull << lane) - 1ull));
    if (keep && slot < n) {
      key[slot] = export_key(jx[job], x0, y0, sg.lg) << kOrderBits | (unsigned)slot;
      fid[slot] = sg.flat_base + (uint32_t)i;
      cnt[slot] = t;
    }
  }
  __syncthreads();
  for (int k = 2; k <= size; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int a = 2 * tid - (tid & (j - 1)), b = a + j;   // the pair's lower place: bit j taken out of tid
      const unsigned long long ka = key[a], kb = key[b];
      if ((ka > kb) == ((a & k) == 0)) {
        key[a] = kb;
        key[b] = ka;
      }
      // pairs up to 64 apart lie in the 128 places of their wave
      const int next = j > 1 ? j >> 1 : k;
      if (j > 64 || next > 64) __syncthreads();
      else wave_sync();
    }
  // the first atoms of the places 2 tid and 2 tid + 1
  const int p = 2 * tid;
  const int f0 = (int)(key[p] & (kOrderMax - 1)), f1 = (int)(key[p + 1] & (kOrderMax - 1));
  const int t0 = p < n ? cnt[f0] : 0, t1 = p + 1 < n ? cnt[f1] : 0;
  int x = t0 + t1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) s_wave[wv] = x;
  __syncthreads();
  int o = x - t0 - t1;
  for (int w = 0; w < wv; ++w) o += s_wave[w];
  if (p < n) {
    vals[p] = fid[f0];
    off[p] = o;
  }
  if (p + 1 < n) {
    vals[p + 1] = fid[f1];
    off[p + 1] = o + t0;
  }
}

// One wave per node in sorted order: its record, then its atoms at the
// scanned offset.
__global__ __launch_bounds__(256) void k_export_write(const ExportSeg* segs, int nseg, const uint32_t* vals,
                                                      const int64_t* off, int64_t n, aqmp_leaf* out,
                                                      int32_t* idx, double* coef) {
  const int lane = threadIdx.x & 63;
  for (int64_t p = blockIdx.x * 4ll + (threadIdx.x >> 6); p < n; p += (int64_t)gridDim.x * 4) {
    const uint32_t fid = vals[p];
    const ExportSeg& sg = segs[seg_of(segs, nseg, fid)];
    const int64_t i = fid - sg.flat_base;
    const int t = sg.L.t[i];
    const int64_t o = off[p];
    if (lane == 0) {
      aqmp_leaf r;
      r.job = sg.L.job[i];
      r.x0 = sg.L.x0[i];
      r.y0 = sg.L.y0[i];
      r.n = 1 << sg.lg;
      r.n_atoms = t;
      r.flags = (sg.L.st[i] & ST_SPLIT) ? 1 : 0;
      r.atom_off = o;
      r.resid_sq = sg.L.e[i];
      out[p] = r;
    }
    const size_t rs = (size_t)i * sg.L.kmax;
    for (int r = lane; r < t; r += 64) {
      idx[o + r] = sg.L.rec_idx[rs + r];
      coef[o + r] = sg.L.rec_coef[rs + r];
    }
  }
}

int grid_1d(int64_t items, int per_block) {
  const int64_t b = (items + per_block - 1) / per_block;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, 4096));
}

}  // namespace

hipError_t launch_export_stats(const ExportSeg* segs, int nseg, int64_t max_cap, ExportTotals* tot, hipStream_t s) {
  if (nseg <= 0) return hipSuccess;
  const dim3 grid(std::min(grid_1d(max_cap, 1024), 64), nseg);
  hipLaunchKernelGGL(k_export_stats, grid, dim3(256), 0, s, segs, tot);
  return hipGetLastError();
}

hipError_t launch_export_keys(const ExportSeg* segs, int nseg, int64_t max_cap, const ExportJob* jx, bool leaves_only,
                              unsigned long long* keys, uint32_t* vals, unsigned long long* next, hipStream_t s) {
  if (nseg <= 0) return hipSuccess;
  const dim3 grid(grid_1d(max_cap, 256), nseg);
  hipLaunchKernelGGL(k_export_keys, grid, dim3(256), 0, s, segs, jx, leaves_only ? 1 : 0, keys, vals, next);
  return hipGetLastError();
}

hipError_t export_sort(void* tmp, size_t& tmp_bytes, unsigned long long* keys, unsigned long long* keys_out,
                       uint32_t* vals, uint32_t* vals_out, int64_t n, int end_bit, hipStream_t s) {
  return rocprim::radix_sort_pairs(tmp, tmp_bytes, keys, keys_out, vals, vals_out, (size_t)n, 0u,
                                   (unsigned)end_bit, s);
}

hipError_t export_scan(void* tmp, size_t& tmp_bytes, const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
  return rocprim::exclusive_scan(tmp, tmp_bytes, in, out, (int64_t)0, (size_t)n, rocprim::plus<int64_t>(), s);
}

hipError_t launch_export_counts(const ExportSeg* segs, int nseg, const uint32_t* vals, int64_t n, int64_t* t_out,
                                hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_export_counts, dim3(grid_1d(n, 256)), dim3(256), 0, s, segs, nseg, vals, n, t_out);
  return hipGetLastError();
}

hipError_t launch_export_order(const ExportSeg* segs, int nseg, const ExportJob* jx, bool leaves_only, int64_t visited,
                               int64_t n, uint32_t* vals, int64_t* off, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n > kOrderMax || nseg > kOrderSegs || visited > kOrderVisited) return hipErrorInvalidValue;
  int size = 128;
  while (size < n) size *= 2;
  hipLaunchKernelGGL(k_export_order, dim3(1), dim3(size / 2), 0, s, segs, nseg, jx, leaves_only ? 1 : 0, (int)visited,
                     (int)n, size, vals, off);
  return hipGetLastError();
}

hipError_t launch_export_write(const ExportSeg* segs, int nseg, const uint32_t* vals, const int64_t* off, int64_t n,
                               aqmp_leaf* out, int32_t* idx, double* coef, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_export_write, dim3(grid_1d(n, 4)), dim3(256), 0, s, segs, nseg, vals, off, n, out, idx,
                     coef);
  return hipGetLastError();
}

}  // namespace aqmp
