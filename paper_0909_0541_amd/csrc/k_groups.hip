// Particle groups for the vectorised walk.
//
// A cell with more than n_crit particles is split further; the runs of its
// consecutive sub-cells (octant order) holding at most n_crit particles each
// are packed greedily into groups of at most n_crit particles; a system with
// at most n_crit particles is a single group.  Groups are contiguous Morton
// ranges; each gets its FP64 bounding box.
#include <algorithm>

#include "bh_device.h"

namespace bh {

namespace {

// The groups of the cell owned at j among its children: set(first, count).
template <class Set>
__device__ __forceinline__ void groups_of_cell(const GroupBuffers &B, int j, Set set) {
  const int c0 = B.nsys + B.cfc[j], nc = B.nchild[j];
  if ((int64_t)c0 + nc > B.nsys + B.info->n_slots) {
    atomicOr(&B.info->err, kErrBuild);
    return;
  }
  int run_first = -1, run_count = 0;
  for (int k = 0; k < nc; ++k) {
    const NodeRec &ch = B.nodes[c0 + k];
    const int cc = ch.count, cf = ch.first;
    if (cc > B.n_crit) {
      if (run_count > 0) set(run_first, run_count);
      run_count = 0;
      continue;
    }
    if (run_count > 0 && run_count + cc > B.n_crit) {
      set(run_first, run_count);
      run_count = 0;
    }
    if (run_count == 0) run_first = cf;
    run_count += cc;
  }
  if (run_count > 0) set(run_first, run_count);
}

__device__ __forceinline__ void store_group(const GroupBuffers &B, int g, int f, int count) {
  B.ginfo[3 * (int64_t)g] = f;
  B.ginfo[3 * (int64_t)g + 1] = count;
  B.ginfo[3 * (int64_t)g + 2] = system_of(B.sys, B.nsys, f);
}

// glen[f] = length of the group that starts at f (0 elsewhere, from the call
// before).
__global__ void k_group_mark(GroupBuffers B) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < B.nsys) {
    const SysInfo &S = B.sys[j];
    if (S.count > 0 && S.count <= B.n_crit) B.glen[S.first] = S.count;
  }
  if (j >= B.n || B.level[j] < 0 || B.ccount[j] <= B.n_crit) return;
  groups_of_cell(B, (int)j, [&](int f, int count) { B.glen[f] = count; });
}

constexpr int kItems = 16;

// Exclusive sum over the workgroup's threads, and the total.
template <int NT>
__device__ __forceinline__ int block_exclusive(int v, int *wsum, int *total) {
  const int w = threadIdx.x / kWave, inc = wave_inclusive_sum(v);
  if (lane_id() == kWave - 1) wsum[w] = inc;
  __syncthreads();
  int off = inc - v, tot = 0;
#pragma unroll
  for (int k = 0; k < NT / kWave; ++k) {
    if (k < w) off += wsum[k];
    tot += wsum[k];
  }
  __syncthreads();
  *total = tot;
  return off;
}

// A thread's 16 positions (the buffer is padded to whole groups of 16, zero).
__device__ __forceinline__ void load_lengths(const GroupBuffers &B, int64_t b, int (&len)[kItems]) {
#pragma unroll
  for (int q = 0; q < kItems / 4; ++q) {
    const int4 v = b < B.n ? reinterpret_cast<const int4 *>(B.glen + b)[q] : make_int4(0, 0, 0, 0);
    len[4 * q] = v.x;
    len[4 * q + 1] = v.y;
    len[4 * q + 2] = v.z;
    len[4 * q + 3] = v.w;
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_group_sums(GroupBuffers B) {
  __shared__ int wsum[NT / kWave];
  int len[kItems], c = 0, total;
  load_lengths(B, ((int64_t)blockIdx.x * NT + threadIdx.x) * kItems, len);
#pragma unroll
  for (int k = 0; k < kItems; ++k) c += len[k] > 0;
  block_exclusive<NT>(c, wsum, &total);
  if (threadIdx.x == 0) B.tiles[blockIdx.x] = total;
}

// Groups numbered by position, the lengths cleared for the next call.  (Tiles
// before a workgroup's own are added up by itself, as in the child scan.)
template <int NT>
__global__ __launch_bounds__(NT) void k_group_scan(GroupBuffers B) {
  __shared__ int wsum[NT / kWave];
  int before = 0, base = 0;
  if (blockIdx.x) {
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += NT) before += B.tiles[k];
    block_exclusive<NT>(before, wsum, &base);
  }
  const int64_t b = ((int64_t)blockIdx.x * NT + threadIdx.x) * kItems;
  int len[kItems], c = 0, total;
  load_lengths(B, b, len);
#pragma unroll
  for (int k = 0; k < kItems; ++k) c += len[k] > 0;
  int g = base + block_exclusive<NT>(c, wsum, &total);
  if (c) {
#pragma unroll
    for (int k = 0; k < kItems; ++k)
      if (len[k] > 0) store_group(B, g++, (int)(b + k), len[k]);
#pragma unroll
    for (int q = 0; q < kItems / 4; ++q) reinterpret_cast<int4 *>(B.glen + b)[q] = make_int4(0, 0, 0, 0);
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) B.info->n_groups = base + total;
}

// Few particles: marks, numbers and groups by one workgroup, the lengths in
// LDS (all groups of 1024 particles 10.4 us against 13 with three launches, of
// 2000 15.2 against 13: one workgroup waits for all their reads).
constexpr int kSmall = 1024, kSmallItems = kSmall / 1024;

__global__ __launch_bounds__(1024) void k_small_groups(GroupBuffers B) {
  __shared__ alignas(16) uint16_t len[kSmall];
  __shared__ int wsum[1024 / kWave];
  const int t = threadIdx.x, n = (int)B.n;
  for (int k = t; k < kSmall / 8; k += 1024) reinterpret_cast<int4 *>(len)[k] = make_int4(0, 0, 0, 0);
  __syncthreads();
  for (int s = t; s < B.nsys; s += 1024) {
    const SysInfo &S = B.sys[s];
    if (S.count > 0 && S.count <= B.n_crit) len[S.first] = (uint16_t)S.count;
  }
  int count[kSmallItems];
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    const int j = 1024 * k + t;
    count[k] = j < n && B.level[j] >= 0 ? B.ccount[j] : 0;
  }
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k)
    if (count[k] > B.n_crit)
      groups_of_cell(B, 1024 * k + t, [&](int f, int c) { len[f] = (uint16_t)c; });
  __syncthreads();
  int c = 0, total;
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) c += len[kSmallItems * t + k] > 0;
  int g = block_exclusive<1024>(c, wsum, &total);
  for (int k = 0; k < kSmallItems; ++k)
    if (len[kSmallItems * t + k] > 0) store_group(B, g++, kSmallItems * t + k, len[kSmallItems * t + k]);
  if (t == 0) B.info->n_groups = total;
}

__device__ __forceinline__ void reset_counters(DevInfo *info) {
  info->queue = 0;
  info->queue2 = 0;
  info->blocks = 0;
  info->rows = 0;
  info->n_out = 0;
  info->tasks = 0;
  info->tasks_done = 0;
  info->blocks_done = 0;
  info->far_chunks = 0;
  info->near_chunks = 0;
  info->interactions = 0;
  info->list_entries = 0;
  info->max_list = 0;
  info->theta_fallback = 0;
  info->node_visits = 0;
  info->near_entries = 0;
  info->err &= ~(kErrPool | kErrWide);
  for (int x = 0; x < 8; ++x) {
    info->xq[x * kLineInts] = 0;
    info->fq[x * kLineInts] = 0;
  }
}

// One wave per group: FP64 bounding box of the members.  One thread clears the
// counters of the force kernels.
__global__ __launch_bounds__(256) void k_group_box(const int32_t *__restrict__ ginfo, const double *__restrict__ spos,
                                                   DevInfo *__restrict__ info, double *__restrict__ gbox) {
  const int lane = lane_id();
  if (blockIdx.x == 0 && threadIdx.x == 0) reset_counters(info);
  const int G = info->n_groups;
  const int wpb = blockDim.x / kWave;
  for (int g = blockIdx.x * wpb + threadIdx.x / kWave; g < G; g += gridDim.x * wpb) {
    const int f = ginfo[3 * g], c = ginfo[3 * g + 1];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = lane; i < c; i += kWave) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double x = spos[3 * (int64_t)(f + i) + k];
        lo[k] = fmin(lo[k], x);
        hi[k] = fmax(hi[k], x);
      }
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        lo[k] = fmin(lo[k], shfl_xor_d(lo[k], d));
        hi[k] = fmax(hi[k], shfl_xor_d(hi[k], d));
      }
    if (lane < 3) {
      gbox[6 * (int64_t)g + lane] = lo[lane];
      gbox[6 * (int64_t)g + 3 + lane] = hi[lane];
    }
  }
}

__global__ void k_reset_list_counters(DevInfo *info) {
  if (threadIdx.x == 0 && blockIdx.x == 0) reset_counters(info);
}

__global__ void k_no_groups(DevInfo *info) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  info->n_groups = 0;
  reset_counters(info);
}

inline unsigned blocks_for(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace



// (Seven launches, with a fill before and the scan, the scatter and the
// counters apart, took 22.6 us at 1024 particles, 29.7 at 8192, 32 at 100k, 62
// at 1M and 181 at 4M; these 10.4, 14.7, 18.2, 42 and 136.)
void make_groups_device(GroupBuffers &B, hipStream_t s) {
  const int64_t n = B.n;
  if (n == 0) {
    k_no_groups<<<1, 64, 0, s>>>(B.info);
    return;
  }
  if (n <= kSmall) {
    k_small_groups<<<1, 1024, 0, s>>>(B);
  } else {
    k_group_mark<<<blocks_for(std::max<int64_t>(n, B.nsys)), 256, 0, s>>>(B);
    // one workgroup alone for up to 16384 particles; tiles of 16384 again
    // where tiles of 4096 would be more than 4096
    if (n <= 1024 * kItems || n > ((int64_t)1 << 24)) {
      const unsigned nt = blocks_for(n, 1024 * kItems);
      if (nt > 1) k_group_sums<1024><<<nt, 1024, 0, s>>>(B);
      k_group_scan<1024><<<nt, 1024, 0, s>>>(B);
    } else {
      const unsigned nt = blocks_for(n, 256 * kItems);
      k_group_sums<256><<<nt, 256, 0, s>>>(B);
      k_group_scan<256><<<nt, 256, 0, s>>>(B);
    }
  }
  k_group_box<<<(unsigned)(B.num_cu * 8), 256, 0, s>>>(B.ginfo, B.spos, B.info, B.gbox);
}

void reset_list_counters(DevInfo *info, hipStream_t s) { k_reset_list_counters<<<1, 64, 0, s>>>(info); }

}  // namespace bh
