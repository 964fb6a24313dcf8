// Oct-tree construction from sorted Morton keys (Sec. 3.1, 3.5).
//
// Cells are identified without pointer chasing.  For neighbouring sorted keys
// i, i+1 of one system let delta_i be the number of leading octal digits they
// share (21 when equal, -1 across a system boundary).  A "split" at i with
// delta_i = l < 21 separates two sub-cells of the level-l cell holding i; the
// cell is owned by its first split (the last particle of its first sub-cell).
// A run of equal keys is a bucket owned by its first particle.  Every other
// prefix with a single non-empty sub-cell is a chain link, which is skipped:
// it holds the same particles as its only child and, for theta < 2/sqrt(3),
// its opening test never accepts it while rejecting the child.
//
// Per-position arrays (index = Morton position) describe the cell owned
// there.  Node records are then placed in slots (k_moments.hip): system roots
// first, the children of every cell in consecutive slots in octant order.
#include <algorithm>

#include "bh_device.h"

namespace bh {

namespace {

// ---------------------------------------------------------------------------
// root cube per system
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_bbox_partial(const double *__restrict__ pos, const SysInfo *__restrict__ sys,
                                                      int bps, double *__restrict__ part, DevInfo *info) {
  __shared__ double red[6][256];
  const int s = blockIdx.x / bps, b = blockIdx.x % bps;
  const int64_t first = sys[s].first, end = first + sys[s].count;
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false;
  for (int64_t i = first + (int64_t)b * blockDim.x + threadIdx.x; i < end; i += (int64_t)bps * blockDim.x) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double x = pos[3 * i + k];
      bad |= !isfinite(x);
      mn[k] = fmin(mn[k], x);
      mx[k] = fmax(mx[k], x);
    }
  }
  if (bad) atomicOr(&info->err, kErrNonFinitePos);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    red[k][threadIdx.x] = mn[k];
    red[3 + k][threadIdx.x] = mx[k];
  }
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        red[k][threadIdx.x] = fmin(red[k][threadIdx.x], red[k][threadIdx.x + w]);
        red[3 + k][threadIdx.x] = fmax(red[3 + k][threadIdx.x], red[3 + k][threadIdx.x + w]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[6 * (int64_t)blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// Root cube from the per-axis extrema: corner at the minimum, side = largest
// extent widened by 2^-20 (1 if all points coincide).
struct Frame {
  double lo[3], side, scale;
};
__device__ __forceinline__ Frame root_frame(const double (&mn)[3], const double (&mx)[3], bool empty) {
  Frame f;
  double ext = 0.0;
  for (int k = 0; k < 3; ++k) {
    f.lo[k] = mn[k];
    const double e = mx[k] - mn[k];
    if (e > ext) ext = e;
  }
  if (empty || !isfinite(ext)) {
    f.lo[0] = f.lo[1] = f.lo[2] = 0.0;
    ext = 0.0;
  }
  f.side = (ext > 0.0) ? __dmul_rn(ext, 1.0 + 0x1p-20) : 1.0;
  f.scale = 0x1p21 / f.side;
  return f;
}

__global__ __launch_bounds__(256) void k_bbox_final(const double *__restrict__ part, int bps, SysInfo *sys) {
  __shared__ double red[6][256];
  const int s = blockIdx.x;
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int b = threadIdx.x; b < bps; b += blockDim.x)
    for (int k = 0; k < 3; ++k) {
      mn[k] = fmin(mn[k], part[6 * ((int64_t)s * bps + b) + k]);
      mx[k] = fmax(mx[k], part[6 * ((int64_t)s * bps + b) + 3 + k]);
    }
  for (int k = 0; k < 3; ++k) {
    red[k][threadIdx.x] = mn[k];
    red[3 + k][threadIdx.x] = mx[k];
  }
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int k = 0; k < 3; ++k) {
        red[k][threadIdx.x] = fmin(red[k][threadIdx.x], red[k][threadIdx.x + w]);
        red[3 + k][threadIdx.x] = fmax(red[3 + k][threadIdx.x], red[3 + k][threadIdx.x + w]);
      }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const double mnv[3] = {red[0][0], red[1][0], red[2][0]}, mxv[3] = {red[3][0], red[4][0], red[5][0]};
  const Frame f = root_frame(mnv, mxv, sys[s].count == 0);
  for (int k = 0; k < 3; ++k) sys[s].lo[k] = f.lo[k];
  sys[s].side = f.side;
  sys[s].scale = f.scale;
}

// ---------------------------------------------------------------------------
// keys
// ---------------------------------------------------------------------------

__global__ void k_system_of_input(const SysInfo *__restrict__ sys, int nsys, int64_t n, int32_t *__restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = system_of(sys, nsys, (int)i);
}

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1fffffu;
  x = (x | (x << 32)) & 0x1f00000000ffffull;
  x = (x | (x << 16)) & 0x1f0000ff0000ffull;
  x = (x | (x << 8)) & 0x100f00f00f00f00full;
  x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

// Peano-Hilbert order (the transposed-index construction of J. Skilling,
// 2004): from the top bit down, the lower bits of x are inverted where an
// axis has the current bit set, and exchanged between x and that axis where
// it has not; a Gray decode across the axes then gives the "transpose" of
// the index, whose bits interleaved level by level (x first) are the index.
// Consecutive indices are face-adjacent cells and every aligned cube is one
// contiguous index range, so the octal digits still name the octree's cells.
__device__ __forceinline__ void hilbert_transpose(uint32_t (&x)[3]) {
  for (int b = kKeyLevels - 1; b >= 1; --b) {
    const uint32_t bit = 1u << b, low = bit - 1u;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const bool set = (x[a] & bit) != 0u;
      const uint32_t sw = (x[0] ^ x[a]) & low;  // (0 for the x axis itself)
      x[0] ^= set ? low : sw;
      x[a] ^= set ? 0u : sw;
    }
  }
  x[1] ^= x[0];
  x[2] ^= x[1];
  uint32_t flip = 0u;
  for (int b = kKeyLevels - 1; b >= 1; --b)
    if (x[2] & (1u << b)) flip ^= (1u << b) - 1u;
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] ^= flip;
}

// Key of a position; the x bit is the most significant of each octal digit.
__device__ __forceinline__ uint64_t cell_key(const double (&x)[3], const double (&lo)[3], double scale, int curve) {
  uint32_t q[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) q[k] = quantise(x[k], lo[k], scale);
  if (curve) hilbert_transpose(q);
  return (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
}

__global__ void k_keys(const double *__restrict__ pos, const double *__restrict__ mass, int64_t n,
                       const int32_t *__restrict__ sys_in, const SysInfo *__restrict__ sys, int curve,
                       uint64_t *__restrict__ keys, uint32_t *__restrict__ vals, PosMass *__restrict__ pm,
                       DevInfo *info) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const SysInfo &S = sys[sys_in ? sys_in[i] : 0];
  const double x[3] = {pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]};
  keys[i] = cell_key(x, S.lo, S.scale, curve);
  vals[i] = (uint32_t)i;
  const double m = mass[i];
  PosMass r;
  r.x = x[0];
  r.y = x[1];
  r.z = x[2];
  r.m = m;
  pm[i] = r;
  if (!(m >= 0.0) || !isfinite(m)) atomicOr(&info->err, kErrBadMass);
}

// Sorted copies and the inverse permutation; the octant masks cleared for the
// topology pass.
__global__ void k_gather(const uint32_t *__restrict__ vals,
                         const PosMass *__restrict__ pm, int64_t n, double *__restrict__ spos,
                         double *__restrict__ smass, int32_t *__restrict__ perm, int32_t *__restrict__ mask) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t j = vals[i];
  perm[i] = (int32_t)j;
  const PosMass r = pm[j];
  spos[3 * i] = r.x;
  spos[3 * i + 1] = r.y;
  spos[3 * i + 2] = r.z;
  smass[i] = r.m;
  mask[i] = 0;
}

// ---------------------------------------------------------------------------
// small trees: root cube, keys, sort and gather in one launch
// ---------------------------------------------------------------------------

// One system of at most kSmallMax particles.  Every workgroup reads all
// positions (they fit an L2 many times over), takes the root cube and the keys
// of all of them, and places its own 32 or 64 particles: a particle's
// sorted place is the number of keys below its own, equal keys in input order,
// the same order as the stable radix sort's.  That is n^2 comparisons (67
// million at 8192), but spread over the chip they take less time than two of
// the thirteen launches they replace: each of those is a chain of a few
// microseconds on a handful of compute units whatever its work.  The whole
// build of 8192 particles takes 155 us instead of 280, of 1000 100 instead of
// 197, of 16384 194 instead of 293 (26 us of the 155 are this launch).
constexpr int kSmallThreads = 1024;

__device__ __forceinline__ void reset_counters(DevInfo *info, int t) {
  static_assert(sizeof(DevInfo) % sizeof(int32_t) == 0, "DevInfo is a whole number of words");
  int32_t *w = reinterpret_cast<int32_t *>(info);
  for (int i = t; i < (int)(sizeof(DevInfo) / sizeof(int32_t)); i += kSmallThreads) w[i] = 0;
}

template <int kSmallTile>
__global__ __launch_bounds__(kSmallThreads) void k_small_sort(const double *__restrict__ pos,
                                                              const double *__restrict__ mass, int n, int curve,
                                                              SysInfo *__restrict__ sys, uint64_t *__restrict__ keys,
                                                              double *__restrict__ spos, double *__restrict__ smass,
                                                              int32_t *__restrict__ perm, int32_t *__restrict__ mask,
                                                              DevInfo *info) {
  extern __shared__ uint64_t lkeys[];  // [n rounded up to 64]
  __shared__ double red[6][kSmallThreads / kWave];
  __shared__ int32_t rank[kSmallTile];
  const int t = threadIdx.x, lane = lane_id(), wv = t / kWave;
  constexpr int kWaves = kSmallThreads / kWave;
  // the first workgroup clears the counters and reports bad input
  const bool first = blockIdx.x == 0;
  if (first) {
    reset_counters(info, t);
    __syncthreads();
  }
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false, badm = false;
#pragma unroll 4
  for (int i = t; i < n; i += kSmallThreads) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double x = pos[3 * (int64_t)i + k];
      bad |= !isfinite(x);
      mn[k] = fmin(mn[k], x);
      mx[k] = fmax(mx[k], x);
    }
    if (first) {
      const double m = mass[i];
      badm |= !(m >= 0.0) || !isfinite(m);
    }
  }
  if (first && bad) atomicOr(&info->err, kErrNonFinitePos);
  if (first && badm) atomicOr(&info->err, kErrBadMass);
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      mn[k] = fmin(mn[k], shfl_xor_d(mn[k], d));
      mx[k] = fmax(mx[k], shfl_xor_d(mx[k], d));
    }
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      red[k][wv] = mn[k];
      red[3 + k][wv] = mx[k];
    }
  if (t < kSmallTile) rank[t] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 3; ++k)
    for (int w = 0; w < kWaves; ++w) {
      mn[k] = fmin(mn[k], red[k][w]);
      mx[k] = fmax(mx[k], red[3 + k][w]);
    }
  const Frame f = root_frame(mn, mx, false);
  if (first && t == 0) {
    for (int k = 0; k < 3; ++k) sys[0].lo[k] = f.lo[k];
    sys[0].side = f.side;
    sys[0].scale = f.scale;
  }
  const int np = (n + kWave - 1) / kWave * kWave;
#pragma unroll 2
  for (int i = t; i < np; i += kSmallThreads) {
    uint64_t k = ~0ull;  // (places beyond n: above every key)
    if (i < n) {
      const double x[3] = {pos[3 * (int64_t)i], pos[3 * (int64_t)i + 1], pos[3 * (int64_t)i + 2]};
      k = cell_key(x, f.lo, f.scale, curve);
    }
    lkeys[i] = k;
  }
  __syncthreads();
  // ranks: wave wv against the wv-th part of the keys, in steps of 64 (with 32
  // own keys, each half of the wave against 32 of them)
  const int i0 = blockIdx.x * kSmallTile;
  const int u = lane & (kSmallTile - 1), i = i0 + u;
  const uint64_t ki = lkeys[min(i, np - 1)];
  int r = 0;
  for (int jw = wv * kWave; jw < np; jw += kSmallThreads) {
    const int j0 = jw + (kSmallTile < kWave ? lane & kSmallTile : 0);
    if (j0 != i0) {  // (the keys lie before, after or on the workgroup's own)
      const uint64_t top = j0 < i0 ? ki + 1 : ki;  // equal keys before: below
#pragma unroll 16
      for (int j = 0; j < kSmallTile; ++j) r += lkeys[j0 + j] < top ? 1 : 0;
    } else {
      for (int j = 0; j < kSmallTile; ++j) {
        const uint64_t kj = lkeys[j0 + j];
        r += (kj < ki || (kj == ki && j < u)) ? 1 : 0;
      }
    }
  }
  if (r) atomicAdd(&rank[u], r);
  __syncthreads();
  if (t >= kSmallTile || i >= n) return;
  const int p = rank[t];
  keys[p] = ki;
  perm[p] = i;
  mask[p] = 0;
  smass[p] = mass[i];
#pragma unroll
  for (int k = 0; k < 3; ++k) spos[3 * (int64_t)p + k] = pos[3 * (int64_t)i + k];
}

// ---------------------------------------------------------------------------
// topology
// ---------------------------------------------------------------------------

// owner[j]: the owning position of the cell split at j (its first split), or
// the first particle of the run of equal keys containing j; level[j]: level
// of the cell owned at j, -1 when j owns none; for an owned cell also its
// particle range (cfirst, ccount).  delta[j]: the split depth of j and j + 1
// (-1 across a system boundary or at the end).
__global__ void k_owner(const uint64_t *__restrict__ keys, int8_t *__restrict__ delta, int64_t n,
                        const SysInfo *__restrict__ sys, int nsys, int32_t *__restrict__ owner,
                        int8_t *__restrict__ level, int32_t *__restrict__ cfirst, int32_t *__restrict__ ccount) {
  int64_t jj = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (jj >= n) return;
  const int j = (int)jj;
  int own = -1, lev = -1, a = 0, b = -1;
  const int s = system_of(sys, nsys, j);
  const int lo = sys[s].first, hi = lo + sys[s].count;
  const uint64_t kj = keys[j];
  const int d = j + 1 < hi ? common_digits(kj, keys[j + 1]) : -1;
  delta[j] = (int8_t)d;
  if (d >= 0) {
    if (d < kKeyLevels) {
      const int sh = prefix_shift(d);
      a = gallop_first(keys, lo, j, kj >> sh, sh);
      const int sh1 = prefix_shift(d + 1);
      int e = gallop_past(keys, a, j + 1, keys[a] >> sh1, sh1);
      own = e - 1;
      if (own == j) {
        lev = d;
        b = gallop_past(keys, j, hi, kj >> sh, sh) - 1;
      }
    } else {
      own = gallop_first(keys, lo, j, kj, 0);
      if (j == lo || keys[j - 1] != kj) {
        lev = kKeyLevels;
        a = j;
        b = gallop_past(keys, j, hi, kj, 0) - 1;
      }
    }
  }
  owner[j] = own;
  level[j] = (int8_t)lev;
  if (lev >= 0) {
    cfirst[j] = a;
    ccount[j] = b - a + 1;
  }
}

// bit into mask[P] for every active lane of the wave, with one atomic per
// run of neighbouring lanes that share P (neighbouring positions mostly
// share a parent; an OR is the same whatever the grouping).  Every lane of
// the wave must call it.
__device__ __forceinline__ void or_into_parent(int32_t *__restrict__ mask, int P, int bit, bool active) {
  const int lane = lane_id();
  const int key = active ? P : -1;
  // (every lane takes part in the shuffles: a lane left out of one gives 0)
  const int prev = __shfl_up(key, 1, kWave), next = __shfl_down(key, 1, kWave);
  const bool head = lane == 0 || prev != key;
  const int run = __popcll(__ballot(head) & ((2ull << lane) - 1ull));
  int v = active ? bit : 0;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int u = __shfl_up(v, d, kWave);
    const int r = __shfl_up(run, d, kWave);
    if (lane >= d && r == run) v |= u;
  }
  const bool tail = lane == kWave - 1 || next != key;
  if (active && tail && v) atomicOr(&mask[P], v);
}

// Parents: of every owned cell (its octant too) and of every particle (a cell,
// a bucket, or none for a system of one particle); octant masks of the parents;
// classes of the cells for the moments pass (sub, piece: its limits).
__global__ void k_parents(const uint64_t *__restrict__ keys, const int8_t *__restrict__ delta,
                          const int32_t *__restrict__ owner, const int8_t *__restrict__ level, int64_t n,
                          const SysInfo *__restrict__ sys, int nsys, const int32_t *__restrict__ cfirst,
                          const int32_t *__restrict__ ccount, int32_t *__restrict__ cparent,
                          int8_t *__restrict__ cdigit, int32_t *__restrict__ pparent, int8_t *__restrict__ pdigit,
                          int32_t *__restrict__ mask, int sub, int piece, uint8_t *__restrict__ kind) {
  const int64_t jj = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int j = (int)jj;
  const bool live = jj < n;
  const int s = live ? system_of(sys, nsys, j) : 0;
  const int lo = live ? sys[s].first : 0;
  const int l = live ? level[j] : -1;
  int P = -1, bit = 0, kd = 0;
  if (l >= 0) {
    const int c = ccount[j];
    const int a = cfirst[j], b = a + c - 1;
    const int dl = (a > lo) ? delta[a - 1] : -1;
    const int dr = delta[b];
    const int lp = max(dl, dr);
    if (lp < 0) {
      cparent[j] = -1 - s;
      cdigit[j] = 0;
    } else {
      const int sp = (dl == lp) ? a - 1 : b;
      P = owner[sp];
      const int dg = key_digit(keys[a], lp + 1);
      cparent[j] = P;
      cdigit[j] = (int8_t)dg;
      bit = 1 << dg;
    }
    const int cp = P >= 0 ? ccount[P] : INT32_MAX;
    if (c > piece) kd = kClassHigh;
    else if (c > sub) kd = cp > piece ? kClassPiece : kClassTop;
    else if (cp > sub) kd = kClassSub;
    if (l == kKeyLevels) kd |= kKindBucket;
  }
  or_into_parent(mask, P, bit, P >= 0);
  P = -1;
  bit = 0;
  if (live) {
    const int dl = (j > lo) ? delta[j - 1] : -1;
    const int dr = delta[j];
    const int lp = max(dl, dr);
    if (lp < 0) {
      pparent[j] = -1 - s;
      pdigit[j] = 0;
    } else {
      const int sp = (dl == lp) ? j - 1 : j;
      P = owner[sp];
      pparent[j] = P;
      if (lp == kKeyLevels) {
        pdigit[j] = 0;  // bucket member: slot order is Morton order
      } else {
        const int dg = key_digit(keys[j], lp + 1);
        pdigit[j] = (int8_t)dg;
        bit = 1 << dg;
      }
    }
    if (P < 0 || ccount[P] > sub) kd |= kKindLone;
    kind[j] = (uint8_t)kd;
  }
  or_into_parent(mask, P, bit, bit != 0);
}

inline unsigned blocks_for(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

// ---------------------------------------------------------------------------
// host-side driver of the build
// ---------------------------------------------------------------------------



int bbox_blocks_per_system(int nsys) {
  int bps = 1024 / (nsys > 0 ? nsys : 1);
  return bps < 4 ? 4 : bps;
}

template <int TILE>
static void launch_small(TreeBuffers &B, hipStream_t s) {
  const int n = (int)B.n;
  const size_t lds = sizeof(uint64_t) * (size_t)((n + kWave - 1) / kWave * kWave);
  k_small_sort<TILE><<<(unsigned)((n + TILE - 1) / TILE), kSmallThreads, lds, s>>>(
      B.pos, B.mass, n, B.curve, B.sys, B.keys[0], B.spos, B.smass, B.perm, B.mask, B.info);
}

// Root cube, keys and the particles in key order.
static const uint64_t *sort_particles(TreeBuffers &B, hipStream_t s) {
  const int64_t n = B.n;
  const int nsys = B.nsys;
  if (nsys == 1 && n <= kSmallMax) {
    // 32 keys per workgroup while they all run at once (a compute unit holds
    // two with up to 64 KiB of keys), 64 beyond
    if (n <= 8192)
      launch_small<32>(B, s);
    else
      launch_small<64>(B, s);
    return B.keys[0];
  }
  reset_info_device(B.info, s);
  const int bps = bbox_blocks_per_system(nsys);
  k_bbox_partial<<<(unsigned)(nsys * bps), 256, 0, s>>>(B.pos, B.sys, bps, B.bbox_part, B.info);
  k_bbox_final<<<(unsigned)nsys, 256, 0, s>>>(B.bbox_part, bps, B.sys);
  if (nsys > 1) k_system_of_input<<<blocks_for(n), 256, 0, s>>>(B.sys, nsys, n, B.sys_in);
  k_keys<<<blocks_for(n), 256, 0, s>>>(B.pos, B.mass, n, nsys > 1 ? B.sys_in : nullptr, B.sys, B.curve, B.keys[0],
                                        B.vals[0], B.pm, B.info);
  int cur = radix_sort_pairs(B.keys[0], B.keys[1], B.vals[0], B.vals[1], n, 0, 64, B.hist, B.scan_tmp,
                             &B.info->err, s);
  if (nsys > 1) {
    for (int shift = 0; (nsys - 1) >> shift; shift += 8)
      cur = radix_pass_by_system(B.keys[0], B.keys[1], B.vals[0], B.vals[1], cur, n, B.sys_in, shift, B.hist,
                                 B.scan_tmp, s);
  }
  k_gather<<<blocks_for(n), 256, 0, s>>>(B.vals[cur], B.pm, n, B.spos, B.smass, B.perm, B.mask);
  return B.keys[cur];
}

void build_tree_device(TreeBuffers &B, hipStream_t s) {
  const int64_t n = B.n;
  const int nsys = B.nsys;
  if (n == 0) {
    reset_info_device(B.info, s);
    const int bps = bbox_blocks_per_system(nsys);
    k_bbox_partial<<<(unsigned)(nsys * bps), 256, 0, s>>>(B.pos, B.sys, bps, B.bbox_part, B.info);
    k_bbox_final<<<(unsigned)nsys, 256, 0, s>>>(B.bbox_part, bps, B.sys);
    B.sorted_keys = B.keys[0];
    empty_roots_device(B, s);
    return;
  }
  const uint64_t *keys = sort_particles(B, s);
  B.sorted_keys = const_cast<uint64_t *>(keys);
  k_owner<<<blocks_for(n), 256, 0, s>>>(keys, B.delta, n, B.sys, nsys, B.owner, B.level, B.cfirst, B.ccount);
  k_parents<<<blocks_for(n), 256, 0, s>>>(keys, B.delta, B.owner, B.level, n, B.sys, nsys, B.cfirst, B.ccount,
                                           B.cparent, B.cdigit, B.pparent, B.pdigit, B.mask,
                                           subtree_particles(n, B.qmom != nullptr, B.largest),
                                           piece_particles(n, B.qmom != nullptr, B.largest), B.kind);
  moments_device(B, s);
}

}  // namespace bh
