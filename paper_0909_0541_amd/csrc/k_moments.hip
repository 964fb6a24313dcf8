// Slots and moments of the tree's nodes (Sec. 3.1, Eq. 2/3).
//
// The children of every cell occupy consecutive slots, given by a scan of the
// child counts over the cells' owning positions.  The moments of a cell are
// its children's raw sums (m, m x, m y, m z) added in slot order starting from
// zero, so the FP64 sums are exactly those of a recursive evaluation.
//
// A level needs the one below it, so a cell costs one step of a serial chain;
// what a step costs decides.  Cells of at most kSub particles hold all but a
// few thousand of the nodes.  The largest of them (subtrees: their parents
// hold more) are handled by one workgroup each (k_subtrees): a subtree's
// particles are consecutive, its cells are owned by positions among them and
// their children fill consecutive slots, so topology and sums live in LDS, a
// level costs an LDS round and a barrier, and divisions, square roots and
// record writes come afterwards for all cells at once.  The cells above are
// taken the same way in pieces (k_top_cells): those under cells of at most
// kFan subtree sizes by a workgroup each, the rest by one.
#include <algorithm>

#include "bh_device.h"

namespace bh {

namespace {

constexpr int kScanItems = 16;

// Offsets or totals of the lists of the child scan.
struct Counts {
  int v[5];  // children; subtrees; pieces of cells above them; their cells; cells above the pieces
};

// What the cell owned at a position (its class in k) adds to them.
__device__ __forceinline__ Counts cell_counts(int k, int children) {
  const int c = k & kClassMask;
  return {{children, c == kClassSub, c == kClassPiece, c == kClassPiece || c == kClassTop, c == kClassHigh}};
}

// Exclusive sums over the workgroup's threads, and the total.
template <int NT>
__device__ __forceinline__ Counts block_exclusive(const Counts &c, int (*wsum)[5], Counts *total) {
  const int w = threadIdx.x / kWave;
  Counts inc, off;
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    inc.v[q] = wave_inclusive_sum(c.v[q]);
    off.v[q] = inc.v[q] - c.v[q];
    total->v[q] = 0;
    if (lane_id() == kWave - 1) wsum[w][q] = inc.v[q];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NT / kWave; ++k)
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const int s = wsum[k][q];
      if (k < w) off.v[q] += s;
      total->v[q] += s;
    }
  __syncthreads();
  return off;
}

// Children of the cells owned at 16 consecutive positions, and their classes.
__device__ __forceinline__ void load_cells(const MomentArgs &a, int64_t b, uint32_t (&kind)[4], int (&nc)[kScanItems]) {
  // (the buffers are padded to whole groups of 16)
  const int4 *mk = reinterpret_cast<const int4 *>(a.mask + b);
  const uint4 kd = *reinterpret_cast<const uint4 *>(a.kind + b);
  kind[0] = kd.x;
  kind[1] = kd.y;
  kind[2] = kd.z;
  kind[3] = kd.w;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int4 m = mk[q];
    nc[4 * q] = __popc(m.x);
    nc[4 * q + 1] = __popc(m.y);
    nc[4 * q + 2] = __popc(m.z);
    nc[4 * q + 3] = __popc(m.w);
  }
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const int64_t j = b + q;
    const int k = (kind[q / 4] >> (8 * (q % 4))) & 255;
    if (j >= a.n) {
      nc[q] = 0;
      kind[q / 4] &= ~(255u << (8 * (q % 4)));
    } else if (k & kKindBucket) {
      nc[q] = a.ccount[j];
    }
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_child_sums(MomentArgs a) {
  __shared__ int wsum[NT / kWave][5];
  const int64_t b = ((int64_t)blockIdx.x * NT + threadIdx.x) * kScanItems;
  Counts s{}, tot;
  if (b < a.n) {
    uint32_t kind[4];
    int nc[kScanItems];
    load_cells(a, b, kind, nc);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const Counts c = cell_counts(kind[k / 4] >> (8 * (k % 4)), nc[k]);
#pragma unroll
      for (int q = 0; q < 5; ++q) s.v[q] += c.v[q];
    }
  }
  block_exclusive<NT>(s, wsum, &tot);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 5; ++q) a.tiles[8 * (int64_t)blockIdx.x + q] = tot.v[q];
}

// First child of every cell (exclusive sum of the child counts), and the lists
// in position order.  A workgroup adds up the sums of the tiles before its own
// (reading at most a few thousand: the host takes longer tiles for more
// particles), so one launch ends the scan.
template <int NT>
__global__ __launch_bounds__(NT) void k_child_scan(MomentArgs a) {
  __shared__ int wsum[NT / kWave][5];
  Counts before{}, off0{};
  if (blockIdx.x) {
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += NT)
#pragma unroll
      for (int q = 0; q < 5; ++q) before.v[q] += a.tiles[8 * (int64_t)k + q];
    block_exclusive<NT>(before, wsum, &off0);
  }
  const int64_t b = ((int64_t)blockIdx.x * NT + threadIdx.x) * kScanItems;
  uint32_t kind[4] = {0, 0, 0, 0};
  int nc[kScanItems];
  Counts s{}, tot;
  if (b < a.n) {
    load_cells(a, b, kind, nc);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const Counts c = cell_counts(kind[k / 4] >> (8 * (k % 4)), nc[k]);
#pragma unroll
      for (int q = 0; q < 5; ++q) s.v[q] += c.v[q];
    }
  }
  Counts off = block_exclusive<NT>(s, wsum, &tot);
#pragma unroll
  for (int q = 0; q < 5; ++q) off.v[q] += off0.v[q];
  if (b < a.n) {
    int fc[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int32_t j = (int32_t)(b + k);
      const Counts c = cell_counts(kind[k / 4] >> (8 * (k % 4)), nc[k]);
      fc[k] = off.v[0];
      if (c.v[1]) a.subs[off.v[1]] = j;
      if (c.v[2]) a.pieces[off.v[2]] = off.v[3];
      if (c.v[3]) a.tops[off.v[3]] = j;
      if (c.v[4]) a.highs[off.v[4]] = j;
#pragma unroll
      for (int q = 0; q < 5; ++q) off.v[q] += c.v[q];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      reinterpret_cast<int4 *>(a.cfc + b)[q] = make_int4(fc[4 * q], fc[4 * q + 1], fc[4 * q + 2], fc[4 * q + 3]);
      reinterpret_cast<int4 *>(a.nchild + b)[q] = make_int4(nc[4 * q], nc[4 * q + 1], nc[4 * q + 2], nc[4 * q + 3]);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    const int slots = off0.v[0] + tot.v[0];
    a.info->n_slots = slots;
    // every cell and particle but the roots of the non-empty systems is a child
    a.info->n_cells = (int32_t)((int64_t)slots + a.nonempty - a.n);
    a.info->n_subs = off0.v[1] + tot.v[1];
    a.info->n_pieces = off0.v[2] + tot.v[2];
    a.info->n_tops = off0.v[3] + tot.v[3];
    a.info->n_highs = off0.v[4] + tot.v[4];
  }
}

__device__ __forceinline__ int slot_under(int nsys, int cfc, int mask, int dg) {
  return nsys + cfc + __popc(mask & ((1 << dg) - 1));
}

__device__ __forceinline__ bool bad_slot(const MomentArgs &a, int slot) {
  if (slot >= 0 && slot < a.cap) return false;
  atomicOr(&a.info->err, kErrBuild);
  return true;
}

__device__ __forceinline__ void note_level(const MomentArgs &a, int lev) {
  // (only the first few find a shallower one)
  if (lev > __hip_atomic_load(&a.info->max_level, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(&a.info->max_level, lev);
}

// Record of particle j; its raw sums.
__device__ __forceinline__ void leaf_record(const MomentArgs &a, int j, int slot, const double (&x)[3], double m,
                                            double (&sum)[4]) {
  NodeRec r;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    r.com[k] = x[k];
    sum[1 + k] = __dmul_rn(m, x[k]);
  }
  sum[0] = r.m = m;
  r.l = 0.0;
  r.s = 0.0;
  r.child = -1;
  r.nchild = 0;
  r.first = j;
  r.count = 1;
  a.nodes[slot] = r;
  a.meta[slot] = (int8_t)(32 * kParticle + 31);
}

struct CellIds {
  int j, slot, c0, nc, first, count;  // owning position, slots, particles
};

// Record of a cell from its raw sums; its centre of mass.  x: position of the
// particle at the owning position, which lies in the cell; lp: level of the
// parent, -1 for a root.
__device__ __forceinline__ void cell_record(const MomentArgs &a, const SysInfo &S, const CellIds &c, int lev, int lp,
                                            const double (&x)[3], const double (&sum)[4], double (&com)[3]) {
  // A bucket (level 21) is opened unless a chain of single-child cells sits
  // above it: the opening bound shrinks down a chain (theta < 2/sqrt(3)), so
  // the chain is accepted iff its deepest cell, at level 20, is; the bucket
  // then carries that cell's side and s.
  const bool bucket = lev == kKeyLevels, always_open = bucket && lp >= kKeyLevels - 1;
  const int geo = (bucket && !always_open) ? kKeyLevels - 1 : lev;
  // The cell's coordinates at level geo: the top geo bits of each quantised
  // coordinate of any of its members (a cell of either curve is one aligned
  // cube, a bucket one point).
  const double l = ldexp(S.side, -geo);
  double d2 = 0.0;
  NodeRec r;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t q = quantise(x[k], S.lo[k], S.scale) >> (kKeyLevels - geo);
    const double centre = __dadd_rn(S.lo[k], __dmul_rn((double)q + 0.5, l));
    com[k] = (sum[0] > 0.0) ? sum[1 + k] / sum[0] : centre;
    r.com[k] = com[k];
    const double d = __dsub_rn(centre, com[k]);
    d2 = k == 0 ? __dmul_rn(d, d) : __dadd_rn(d2, __dmul_rn(d, d));
  }
  r.m = sum[0];
  r.l = always_open ? INFINITY : l;
  r.s = sqrt(d2);
  r.child = c.c0;
  r.nchild = c.nc;
  r.first = c.first;
  r.count = c.count;
  a.nodes[c.slot] = r;
  a.meta[c.slot] = (int8_t)(bucket ? 32 * kBucket + lev : lev);
  a.cslot[c.j] = c.slot;
}

// A child's part of a cell's second moments about com (parallel axes): its
// own moments (nullptr: a particle's, zero) and its mass mc > 0 at its centre
// of mass c.
__device__ __forceinline__ void shift_moments(double (&S)[6], const double (&com)[3], double mc, const double *c,
                                              const double *own) {
  const double ex = __dsub_rn(c[0], com[0]), ey = __dsub_rn(c[1], com[1]), ez = __dsub_rn(c[2], com[2]);
  const double sh[6] = {mc * ex * ex, mc * ey * ey, mc * ez * ez, mc * ex * ey, mc * ex * ez, mc * ey * ez};
#pragma unroll
  for (int k = 0; k < 6; ++k) S[k] = __dadd_rn(S[k], own ? __dadd_rn(own[k], sh[k]) : sh[k]);
}

// A cell's second moments, and as the force sum reads them: 3 S and the trace
// T (and 1.5 T).
__device__ __forceinline__ void store_moments(const MomentArgs &a, int slot, const double (&S)[6]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) a.qmom[6 * (int64_t)slot + k] = S[k];
  const double T = S[0] + S[1] + S[2];
  a.qpack[2 * (int64_t)slot] = make_float4((float)(3.0 * S[0]), (float)(3.0 * S[1]), (float)(3.0 * S[2]),
                                           (float)(3.0 * S[3]));
  a.qpack[2 * (int64_t)slot + 1] = make_float4((float)(3.0 * S[4]), (float)(3.0 * S[5]), (float)T, (float)(1.5 * T));
}

// Particles of a subtree, and threads of its workgroup (with few particles
// twice as many: up to 1024 of them then are one subtree; the build of 1024
// and 8192 particles 62 and 81 us with 512, 47 and 78 with 1024; of 1M 484 and
// 510).
constexpr int kSub = 512, kSubFew = 1024, kSubQuad = 256;
constexpr int64_t kFewParticles = 16384;
// Largest tree whose second moments are made with its subtrees: builds in us that
// way and with launches by level, clustered boxes of 300k, 500k, 600k, 1M, 4M and
// 8M particles 404, 497, 573, 849, 2421, 4375 and 436, 494, 551, 750, 1966, 3538,
// uniform spheres of 300k, 500k and 600k 328, 394, 560 and 413, 469, 518.
constexpr int64_t kQuadParticles = 1 << 19;
// Batches of at least so many systems take their subtrees of up to 64 particles
// by a wave each: a workgroup of 512 threads for each of 65,536 systems of 4 or 16
// particles made the build 1619 and 1882 us (launches by level 1213 and 1434, now
// 1140 and 1347; 256 systems of 4 139).  And systems of 513 to 1024 particles are
// one subtree each, with nothing above: 4000 of 1000 1557 us, in subtrees of 512
// 1828.
constexpr int kManySystems = 256;

// One workgroup per subtree; afterwards the particles whose parents are above
// the subtrees.  A subtree of c particles at positions [f, f + c) owns its
// cells at positions [f, f + c - 1) (the last position may own an ancestor),
// and their children have the slots from cfc[f] on, at most 2 c - 2.  Bound by
// latency for small trees (subtree, its arrays, levels, records) and by the
// scattered 64-byte records for large ones: 11 us at 8192 particles, 380 us at
// 4M (records and sums read and written once: 150 us).  One launch per tree level over sums in global memory, with
// a pass for the slots and leaves and a counting sort of the cells by level
// before: the whole build of 8192, 100k, 1M and 4M particles 158, 270, 544 and
// 1443 us; with this 78, 198, 481 and 1342 us.  Subtrees of 256 with second
// moments: of 512 (one workgroup a compute unit) took 222 us.  They are bound by
// the workgroups in flight, with moments in LDS for cells only, not leaves, and
// five waves a SIMD (the build of 300k particles 386 us, with room for three
// workgroups 405); larger trees take them level by level (k_second_moments).
//
// With SPLIT a launch takes the subtrees of more than `above` and at most SUB
// particles, one of them (lone) those particles.
template <int SUB, bool QUAD, bool SPLIT>
__global__ __launch_bounds__(SUB) __attribute__((amdgpu_waves_per_eu(QUAD ? 5 : 1))) void k_subtrees(MomentArgs a,
                                                                                                   int above,
                                                                                                   bool lone) {
  constexpr int LOCAL = 2 * SUB, ROOT = LOCAL - 1;
  __shared__ double sm[LOCAL][4];
  __shared__ double qm[QUAD ? SUB : 1][6];   // of the cell owned at a position
  __shared__ int16_t cell[QUAD ? LOCAL : 1];  // that position, -1: a particle
  __shared__ int lcfc[SUB], lmask[SUB];
  __shared__ int8_t llev[SUB];
  __shared__ uint32_t levels;
  const int t = threadIdx.x;
  const int nsub = a.info->n_subs;
  for (int i = blockIdx.x; i < nsub; i += gridDim.x) {
    const int r = a.subs[i];
    const int f = a.cfirst[r], cnt = SPLIT ? a.ccount[r] : min(a.ccount[r], SUB);
    if (SPLIT && (cnt <= above || cnt > SUB)) continue;
    const SysInfo &S = a.sys[system_of(a.sys, a.nsys, f)];
    const int j = f + t;
    if (t == 0) levels = 0;
    // everything of the position at once
    int lev = -1, pp = 0, pd = 0, cp = 0, cd = 0;
    CellIds c{};
    double x[3] = {0.0, 0.0, 0.0}, m = 0.0;
    if (t < cnt) {
      lev = a.level[j];
      pp = a.pparent[j];
      pd = a.pdigit[j];
      cp = a.cparent[j];
      cd = a.cdigit[j];
      c.c0 = a.cfc[j];
      c.nc = a.nchild[j];
      c.first = a.cfirst[j];
      c.count = a.ccount[j];
      const int mk = a.mask[j];
#pragma unroll
      for (int k = 0; k < 3; ++k) x[k] = a.spos[3 * (int64_t)j + k];
      m = a.smass[j];
      lcfc[t] = c.c0;
      lmask[t] = mk;
      llev[t] = (int8_t)lev;
      if (t == cnt - 1) lev = -1;
    }
    c.j = j;
    int lp = -1, rslot = -1;
    if (j == r) {
      rslot = -1 - cp;
      if (cp >= 0) {
        rslot = slot_under(a.nsys, a.cfc[cp], a.mask[cp], cd);
        lp = a.level[cp];
      }
    }
    __syncthreads();
    const int base = a.nsys + lcfc[0];
    double sum[4];
    int leaf = -1;
    if (t < cnt) {
      const int p = pp - f;
      int slot = -1;
      if (p >= 0 && p < cnt)
        slot = llev[p] == kKeyLevels ? a.nsys + lcfc[p] + (t - p)  // bucket member: Morton order
                                     : slot_under(a.nsys, lcfc[p], lmask[p], pd);
      const int at = slot - base;
      if (!bad_slot(a, slot) && at >= 0 && at < ROOT) {
        leaf_record(a, j, slot, x, m, sum);
#pragma unroll
        for (int k = 0; k < 4; ++k) sm[at][k] = sum[k];
        if (QUAD) {
          leaf = at;
          cell[at] = -1;
        }
      }
    }
    int own = ROOT, lc0 = 0;
    if (lev >= 0) {
      c.c0 += a.nsys;
      lc0 = c.c0 - base;
      if (j == r) {
        c.slot = rslot;
      } else {
        const int p = cp - f;
        c.slot = -1;
        if (p >= 0 && p < cnt) {
          c.slot = slot_under(a.nsys, lcfc[p], lmask[p], cd);
          lp = llev[p];
        }
        own = c.slot - base;
      }
      if (bad_slot(a, c.slot) || own < 0 || own > ROOT || lc0 < 0 || c.nc < 0 || lc0 + c.nc > ROOT) {
        atomicOr(&a.info->err, kErrBuild);
        lev = -1;
      }
    }
    {
      uint32_t have = lev >= 0 ? 1u << lev : 0u;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) have |= __shfl_xor(have, d, kWave);
      if (lane_id() == 0 && have) atomicOr(&levels, have);
    }
    __syncthreads();
    const uint32_t all = levels;
    for (uint32_t L = all; L;) {
      const int cur = 31 - __clz(L);
      L &= ~(1u << cur);
      if (lev == cur) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        for (int k = 0; k < c.nc; ++k) {
          const double *h = sm[lc0 + k];
          s0 = __dadd_rn(s0, h[0]);
          s1 = __dadd_rn(s1, h[1]);
          s2 = __dadd_rn(s2, h[2]);
          s3 = __dadd_rn(s3, h[3]);
        }
        sum[0] = sm[own][0] = s0;
        sum[1] = sm[own][1] = s1;
        sum[2] = sm[own][2] = s2;
        sum[3] = sm[own][3] = s3;
      }
      __syncthreads();
    }
    double com[3];
    if (lev >= 0) {
      cell_record(a, S, c, lev, lp, x, sum, com);
      if (own == ROOT)
#pragma unroll
        for (int k = 0; k < 4; ++k) a.msum[4 * (int64_t)c.slot + k] = sum[k];
    }
    if (QUAD) {
      // sums to centres of mass, in place
      if (leaf >= 0 && m > 0.0)
#pragma unroll
        for (int k = 0; k < 3; ++k) sm[leaf][1 + k] /= m;
      if (lev >= 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) sm[own][1 + k] = com[k];
      if (lev >= 0) cell[own] = (int16_t)t;
      __syncthreads();
      double M[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      for (uint32_t L = all; L;) {
        const int cur = 31 - __clz(L);
        L &= ~(1u << cur);
        if (lev == cur) {
          for (int k = 0; k < c.nc; ++k) {
            const double mc = sm[lc0 + k][0];
            const int at = cell[lc0 + k];
            if (mc > 0.0) shift_moments(M, com, mc, &sm[lc0 + k][1], at >= 0 ? qm[at] : nullptr);
          }
#pragma unroll
          for (int k = 0; k < 6; ++k) qm[t][k] = M[k];
        }
        __syncthreads();
      }
      if (lev >= 0) store_moments(a, c.slot, M);
    }
    if (t == 0 && all) note_level(a, 31 - __clz(all));
    __syncthreads();
  }
  if (SPLIT && !lone) return;
  for (int64_t b = ((int64_t)blockIdx.x * SUB + t) * 16; b < a.n; b += (int64_t)gridDim.x * SUB * 16) {
    const uint4 kd = *reinterpret_cast<const uint4 *>(a.kind + b);
    const uint32_t w[4] = {kd.x, kd.y, kd.z, kd.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      for (uint32_t o = w[q] & (0x01010101u * kKindLone); o; o &= o - 1) {
        const int64_t j = b + 4 * q + (__ffs(o) - 1) / 8;
        if (j >= a.n) break;
        const int P = a.pparent[j];
        int slot = -1 - P;
        if (P >= 0)
          slot = a.level[P] == kKeyLevels ? a.nsys + a.cfc[P] + (int)(j - P)
                                          : slot_under(a.nsys, a.cfc[P], a.mask[P], a.pdigit[j]);
        if (bad_slot(a, slot)) continue;
        const double x[3] = {a.spos[3 * j], a.spos[3 * j + 1], a.spos[3 * j + 2]};
        double s[4];
        leaf_record(a, (int)j, slot, x, a.smass[j], s);
#pragma unroll
        for (int k = 0; k < 4; ++k) a.msum[4 * (int64_t)slot + k] = s[k];
      }
    }
  }
}

// Cells above the subtrees.  The tree above a cell of at most kFan * kSub
// particles has fewer than fan cells of more than kSub particles on each of
// the 22 levels.
template <bool QUAD>
struct Piece {
  static constexpr int kFan = QUAD ? 10 : 16;
  static constexpr int kCap = 22 * kFan;
  static constexpr int kThreads = QUAD ? 256 : 384;
  double sum[kCap][8][4];             // the children's raw sums (88 KiB; with second moments 138 KiB)
  double qm[QUAD ? kCap : 1][8][6];   // and second moments
  int32_t pos[kCap];                  // owning positions, ascending
  uint32_t levels;
};

// A child's raw sums and moments in global memory, whose cell may be a bucket
// of many particles.
constexpr int kMomChunk = 4;

__device__ __forceinline__ void sum_children(const MomentArgs &a, int c0, int nc, double (&sum)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) sum[k] = 0.0;
  for (int cb = 0; cb < nc; cb += kMomChunk) {
    // (the children's sums are read together, indices clamped to the last)
    double2 p[kMomChunk], q[kMomChunk];
#pragma unroll
    for (int u = 0; u < kMomChunk; ++u) {
      const double2 *c = reinterpret_cast<const double2 *>(a.msum + 4 * (int64_t)(c0 + min(cb + u, nc - 1)));
      p[u] = c[0];
      q[u] = c[1];
    }
#pragma unroll
    for (int u = 0; u < kMomChunk; ++u) {
      if (cb + u < nc) {
        sum[0] = __dadd_rn(sum[0], p[u].x);
        sum[1] = __dadd_rn(sum[1], p[u].y);
        sum[2] = __dadd_rn(sum[2], q[u].x);
        sum[3] = __dadd_rn(sum[3], q[u].y);
      }
    }
  }
}

__device__ __forceinline__ void moment_children(const MomentArgs &a, int c0, int nc, const double (&com)[3],
                                                double (&M)[6]) {
  for (int c = c0; c < c0 + nc; ++c) {
    const double *q = a.msum + 4 * (int64_t)c;
    const double mc = q[0];
    const bool leaf = (a.meta[c] >> 5) == kParticle;
    const double x[3] = {q[1] / mc, q[2] / mc, q[3] / mc};
    if (mc > 0.0) shift_moments(M, com, mc, x, leaf ? nullptr : a.qmom + 6 * (int64_t)c);
  }
}

// Ids, level, parent's level and position of the cell owned at j.
__device__ __forceinline__ bool load_cell(const MomentArgs &a, int j, CellIds *c, int *lev, int *P, int *lp,
                                          double (&x)[3]) {
  c->j = j;
  *lev = a.level[j];
  *P = a.cparent[j];
  c->c0 = a.nsys + a.cfc[j];
  c->nc = a.nchild[j];
  c->first = a.cfirst[j];
  c->count = a.ccount[j];
#pragma unroll
  for (int k = 0; k < 3; ++k) x[k] = a.spos[3 * (int64_t)j + k];
  *lp = -1;
  c->slot = -1 - *P;
  if (*P >= 0) {
    *lp = a.level[*P];
    c->slot = slot_under(a.nsys, a.cfc[*P], a.mask[*P], a.cdigit[j]);
  }
  if (!bad_slot(a, c->slot) && c->c0 >= 0 && c->nc >= 0 && (int64_t)c->c0 + c->nc <= a.cap) return true;
  atomicOr(&a.info->err, kErrBuild);
  return false;
}

// The cells owned at list[0, count), count <= kCap, one a thread: parents
// among them (or none of the list's), other children's sums in global memory.
template <bool QUAD>
__device__ void piece(const MomentArgs &a, const int32_t *__restrict__ list, int count, Piece<QUAD> &L) {
  const int t = threadIdx.x;
  const bool on = t < count;
  if (on) L.pos[t] = list[t];
  if (t == 0) L.levels = 0;
  __syncthreads();
  CellIds c{};
  int lev = -1, P = -1, lp = -1, up = -1, rank = 0;
  double x[3], sum[4] = {0.0, 0.0, 0.0, 0.0};
  bool wide = false;  // a bucket: more children than a cell has octants
  if (on && load_cell(a, L.pos[t], &c, &lev, &P, &lp, x)) {
    wide = lev == kKeyLevels;
    if (P >= 0) {
      int lo = 0, hi = count - 1;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (L.pos[mid] < P) lo = mid + 1;
        else hi = mid;
      }
      if (L.pos[lo] == P) {
        up = lo;
        rank = min(c.slot - a.nsys - a.cfc[P], 7);
      }
    }
    if (wide) {
      sum_children(a, c.c0, c.nc, sum);
    } else {
      // (a child of the list overwrites what is read for it here)
      const int nc = min(c.nc, 8);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (k < nc) {
          const int64_t h = c.c0 + k;
#pragma unroll
          for (int q = 0; q < 4; ++q) L.sum[t][k][q] = a.msum[4 * h + q];
          if (QUAD) {
            const bool leaf = (a.meta[h] >> 5) == kParticle;
#pragma unroll
            for (int q = 0; q < 6; ++q) L.qm[t][k][q] = leaf ? 0.0 : a.qmom[6 * h + q];
          }
        }
      }
      c.nc = nc;
    }
    atomicOr(&L.levels, 1u << lev);
  } else {
    lev = -1;
  }
  __syncthreads();
  const uint32_t all = L.levels;
  for (uint32_t m = all; m;) {
    const int cur = 31 - __clz(m);
    m &= ~(1u << cur);
    if (lev == cur) {
      if (!wide) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (k < c.nc)
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[q] = __dadd_rn(sum[q], L.sum[t][k][q]);
      }
      if (up >= 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) L.sum[up][rank][q] = sum[q];
      }
    }
    __syncthreads();
  }
  double com[3];
  if (lev >= 0) {
    cell_record(a, a.sys[system_of(a.sys, a.nsys, c.j)], c, lev, lp, x, sum, com);
    if (up < 0)
#pragma unroll
      for (int q = 0; q < 4; ++q) a.msum[4 * (int64_t)c.slot + q] = sum[q];
  }
  if (QUAD) {
    // the children's sums to centres of mass, in place
    if (lev >= 0 && !wide) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k < c.nc)
#pragma unroll
          for (int q = 0; q < 3; ++q) L.sum[t][k][1 + q] /= L.sum[t][k][0];
    }
    double M[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (uint32_t m = all; m;) {
      const int cur = 31 - __clz(m);
      m &= ~(1u << cur);
      if (lev == cur) {
        if (wide) {
          moment_children(a, c.c0, c.nc, com, M);
        } else {
          for (int k = 0; k < c.nc; ++k) {
            const double mc = L.sum[t][k][0];
            if (mc > 0.0) shift_moments(M, com, mc, &L.sum[t][k][1], L.qm[t][k]);
          }
        }
        if (up >= 0) {
#pragma unroll
          for (int q = 0; q < 6; ++q) L.qm[up][rank][q] = M[q];
        }
      }
      __syncthreads();
    }
    if (lev >= 0) store_moments(a, c.slot, M);
  }
  if (t == 0 && all) note_level(a, 31 - __clz(all));
  __syncthreads();
}

// (9 us at 1024 particles, 11 us at 8192, 53 us at 4M.)
// One workgroup per piece: a cell of at most fan * kSub particles under one
// that holds more, and the cells of more than kSub particles below it.  Its
// cells are neighbours in the list of all such cells.
template <bool QUAD>
__global__ __launch_bounds__(Piece<QUAD>::kThreads) void k_top_cells(MomentArgs a) {
  constexpr int CAP = Piece<QUAD>::kCap;
  __shared__ Piece<QUAD> L;
  const int t = threadIdx.x;
  const int n = a.info->n_pieces, ntop = a.info->n_tops;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const int at = a.pieces[i], r = a.tops[at];
    const int f = a.cfirst[r], last = f + a.ccount[r] - 2;
    const int lo = at - 1 - t, hi = at + 1 + t;
    const int before = __syncthreads_count(t < CAP && lo >= 0 && a.tops[max(lo, 0)] >= f);
    const int after = __syncthreads_count(t < CAP && hi < ntop && a.tops[min(hi, ntop - 1)] <= last);
    const int count = before + after + 1;
    if (count > CAP) {
      if (t == 0) atomicOr(&a.info->err, kErrBuild);
      continue;
    }
    piece<QUAD>(a, a.tops + (at - before), count, L);
  }
}

// The cells above the pieces, by one workgroup: as one more piece if they are
// few, otherwise ordered by level (a counting sort; the order within a level
// does not matter) and taken level by level from the sums in global memory.
template <bool QUAD>
__global__ __launch_bounds__(Piece<QUAD>::kThreads) void k_high_cells(MomentArgs a) {
  constexpr int NT = Piece<QUAD>::kThreads;
  __shared__ Piece<QUAD> L;
  __shared__ int32_t count[kKeyLevels + 1], off[kKeyLevels + 2], cursor[kKeyLevels + 1];
  const int t = threadIdx.x;
  const int n = a.info->n_highs;
  if (n <= Piece<QUAD>::kCap) {
    piece<QUAD>(a, a.highs, n, L);
    return;
  }
  if (t <= kKeyLevels) count[t] = 0;
  __syncthreads();
  for (int i = t; i < n; i += NT) atomicAdd(&count[a.level[a.highs[i]]], 1);
  __syncthreads();
  if (t == 0) {
    int s = 0, deepest = 0;
    for (int l = 0; l <= kKeyLevels; ++l) {
      off[l] = cursor[l] = s;
      s += count[l];
      if (count[l]) deepest = l;
    }
    off[kKeyLevels + 1] = s;
    note_level(a, deepest);
  }
  __syncthreads();
  for (int i = t; i < n; i += NT) {
    const int j = a.highs[i];
    a.highs2[atomicAdd(&cursor[a.level[j]], 1)] = j;
  }
  __syncthreads();
  for (int l = kKeyLevels; l >= 0; --l) {
    if (off[l] == off[l + 1]) continue;  // (the whole workgroup)
    for (int i = off[l] + t; i < off[l + 1]; i += NT) {
      CellIds c;
      int lev, P, lp;
      double x[3], sum[4], com[3];
      if (!load_cell(a, a.highs2[i], &c, &lev, &P, &lp, x)) continue;
      sum_children(a, c.c0, c.nc, sum);
#pragma unroll
      for (int k = 0; k < 4; ++k) a.msum[4 * (int64_t)c.slot + k] = sum[k];
      cell_record(a, a.sys[system_of(a.sys, a.nsys, c.j)], c, lev, lp, x, sum, com);
      if (QUAD) {
        double M[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        moment_children(a, c.c0, c.nc, com, M);
        store_moments(a, c.slot, M);
      }
    }
    // this level's sums before the next level's reads
    __threadfence_block();
    __syncthreads();
  }
}

__global__ void k_empty_roots(const SysInfo *__restrict__ sys, int nsys, NodeRec *__restrict__ nodes,
                              double *__restrict__ msum, int8_t *__restrict__ meta) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nsys || sys[s].count != 0) return;
  NodeRec r;
  r.com[0] = r.com[1] = r.com[2] = 0.0;
  r.m = 0.0;
  r.l = 0.0;
  r.s = 0.0;
  r.child = -1;
  r.nchild = 0;
  r.first = sys[s].first;
  r.count = 0;
  nodes[s] = r;
  meta[s] = (int8_t)(32 * kEmpty + 31);
  for (int k = 0; k < 4; ++k) msum[4 * (int64_t)s + k] = 0.0;
}

// Second moments of large trees, in launches by level over the records that the
// monopole passes have written: the cells listed by level (order within a level
// does not matter), then from the deepest level up.  At 1M particles 20 us for the
// list and 230 for the levels, 4 for each empty one and 20 for the fullest.
constexpr int kLevels = kKeyLevels + 1, kLevelTile = 16;  // positions per thread

// Lanes whose cells have this lane's level (l < 0: none), so that counters see
// one atomic per wave and level.
__device__ __forceinline__ unsigned long long level_peers(int l) {
  unsigned long long peers = __ballot(l >= 0);
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    const unsigned long long m = __ballot(l >= 0 && ((l >> b) & 1));
    peers &= ((l >> b) & 1) ? m : ~m;
  }
  return l >= 0 ? peers : 0ull;
}

__global__ __launch_bounds__(256) void k_level_count(MomentArgs a) {
  __shared__ int32_t c[kLevels];
  const int t = threadIdx.x;
  if (t < kLevels) c[t] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * 256 * kLevelTile + t;
#pragma unroll 4
  for (int q = 0; q < kLevelTile; ++q) {
    const int64_t j = base + 256 * q;
    const int l = j < a.n ? a.level[j] : -1;
    const unsigned long long peers = level_peers(l);
    if (l >= 0 && rank_below(peers) == 0) atomicAdd(&c[l], (int)__popcll(peers));
  }
  __syncthreads();
  if (t < kLevels && c[t]) atomicAdd(&a.level_count[t], c[t]);
}

// A level's places follow those of the levels above (the last one's end in
// level_count[64 + level]).
__global__ __launch_bounds__(256) void k_level_lists(MomentArgs a) {
  __shared__ int32_t c[kLevels], base[kLevels];
  const int t = threadIdx.x;
  if (t < kLevels) c[t] = 0;
  __syncthreads();
  const int64_t b0 = (int64_t)blockIdx.x * 256 * kLevelTile + t;
  int lev[kLevelTile], at[kLevelTile];
#pragma unroll
  for (int q = 0; q < kLevelTile; ++q) {
    const int64_t j = b0 + 256 * q;
    lev[q] = j < a.n ? a.level[j] : -1;
    const unsigned long long peers = level_peers(lev[q]);
    const int rank = rank_below(peers);
    int first = 0;
    if (lev[q] >= 0 && rank == 0) first = atomicAdd(&c[lev[q]], (int)__popcll(peers));
    at[q] = __shfl(first, peers ? __ffsll((long long)peers) - 1 : 0, kWave) + rank;
  }
  __syncthreads();
  if (t < kWave) {
    const int count = t < kLevels ? a.level_count[t] : 0, end = wave_inclusive_sum(count);
    if (t < kLevels) {
      if (blockIdx.x == 0) a.level_count[64 + t] = end;
      if (c[t]) base[t] = end - count + atomicAdd(&a.level_count[32 + t], c[t]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kLevelTile; ++q)
    if (lev[q] >= 0) a.by_level[base[lev[q]] + at[q]] = (int32_t)(b0 + 256 * q);
}

// One cell per thread, a level's time the chain of its reads: its children's
// records and moments (a particle's: never written, unused) are neighbours,
// kMomChunk of them read together (indices clamped to the last).
__global__ __launch_bounds__(256) void k_second_moments(MomentArgs a, int lev) {
  const int end = a.level_count[64 + lev], first = end - a.level_count[lev];
  for (int64_t k = first + (int64_t)blockIdx.x * 256 + threadIdx.x; k < end; k += (int64_t)gridDim.x * 256) {
    const int j = a.by_level[k];
    const int slot = a.cslot[j], c0 = a.nsys + a.cfc[j], nc = a.nchild[j];
    if (bad_slot(a, slot)) continue;
    if (c0 < 0 || nc < 1 || (int64_t)c0 + nc > a.cap) {
      atomicOr(&a.info->err, kErrBuild);
      continue;
    }
    const double com[3] = {a.nodes[slot].com[0], a.nodes[slot].com[1], a.nodes[slot].com[2]};
    double M[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int cb = 0; cb < nc; cb += kMomChunk) {
      double x[kMomChunk][3], m[kMomChunk], own[kMomChunk][6];
      bool leaf[kMomChunk];
#pragma unroll
      for (int u = 0; u < kMomChunk; ++u) {
        const int64_t at = c0 + min(cb + u, nc - 1);
        const NodeRec &r = a.nodes[at];
#pragma unroll
        for (int q = 0; q < 6; ++q) own[u][q] = a.qmom[6 * at + q];
#pragma unroll
        for (int q = 0; q < 3; ++q) x[u][q] = r.com[q];
        m[u] = r.m;
        leaf[u] = r.child < 0;
      }
#pragma unroll
      for (int u = 0; u < kMomChunk; ++u) {
        if (cb + u >= nc || !(m[u] > 0.0)) continue;
        // (a particle's centre of mass as from its raw sums, as in the other passes)
        if (leaf[u])
#pragma unroll
          for (int q = 0; q < 3; ++q) x[u][q] = __dmul_rn(m[u], x[u][q]) / m[u];
        shift_moments(M, com, m[u], x[u], leaf[u] ? nullptr : own[u]);
      }
    }
    store_moments(a, slot, M);
  }
}

void second_moments(const MomentArgs &a, hipStream_t s) {
  const unsigned tiles = (unsigned)((a.n + 256 * kLevelTile - 1) / (256 * kLevelTile));
  fill_i32(a.level_count, 0, 64, s);
  k_level_count<<<tiles, 256, 0, s>>>(a);
  k_level_lists<<<tiles, 256, 0, s>>>(a);
  const unsigned grid = (unsigned)std::min<int64_t>((a.n + 255) / 256, 1024);
  for (int lev = kKeyLevels; lev >= 0; --lev) k_second_moments<<<grid, 256, 0, s>>>(a, lev);
}

template <int SUB, bool QUAD>
void launch(const MomentArgs &a, hipStream_t s) {
  // many systems: the smallest subtrees by a wave each
  const int tiny = a.nonempty >= kManySystems ? kWave : 0;
  const bool larger = a.largest > tiny;
  if (tiny)
    k_subtrees<kWave, QUAD, true><<<(unsigned)std::min(a.nonempty, 1 << 14), kWave, 0, s>>>(a, 0, !larger);
  // (a subtree holds 100 to 250 particles, or a system)
  const int64_t subs = std::max<int64_t>((a.n + 127) / 128, tiny ? 0 : a.nonempty);
  const unsigned grid = (unsigned)std::min<int64_t>(subs, 2048);
  if (larger && tiny) k_subtrees<SUB, QUAD, true><<<grid, SUB, 0, s>>>(a, tiny, true);
  if (!tiny) k_subtrees<SUB, QUAD, false><<<grid, SUB, 0, s>>>(a, 0, true);
  if (a.largest > SUB)
    k_top_cells<QUAD><<<(unsigned)std::min<int64_t>((a.n + 1023) / 1024, 1024), Piece<QUAD>::kThreads, 0, s>>>(a);
  if (a.largest > SUB * Piece<QUAD>::kFan) k_high_cells<QUAD><<<1, Piece<QUAD>::kThreads, 0, s>>>(a);
}

}  // namespace

static bool quad_subtrees(int64_t n, bool quad) { return quad && n <= kQuadParticles; }

int subtree_particles(int64_t n, bool quad, int largest) {
  if (quad_subtrees(n, quad)) return kSubQuad;
  return n <= kFewParticles || (largest > kSub && largest <= kSubFew) ? kSubFew : kSub;
}
int piece_particles(int64_t n, bool quad, int largest) {
  return subtree_particles(n, quad, largest) * (quad_subtrees(n, quad) ? Piece<true>::kFan : Piece<false>::kFan);
}

void empty_roots_device(const TreeBuffers &B, hipStream_t s) {
  k_empty_roots<<<(unsigned)((B.nsys + 255) / 256), 256, 0, s>>>(B.sys, B.nsys, B.nodes, B.msum, B.meta);
}

void moments_device(const TreeBuffers &B, hipStream_t s) {
  MomentArgs a{};
  a.n = B.n;
  a.nsys = B.nsys;
  a.nonempty = B.nonempty;
  a.largest = B.largest;
  a.cap = B.slot_cap;
  a.sys = B.sys;
  a.level = B.level;
  a.cdigit = B.cdigit;
  a.pdigit = B.pdigit;
  a.kind = B.kind;
  a.cfirst = B.cfirst;
  a.ccount = B.ccount;
  a.cparent = B.cparent;
  a.pparent = B.pparent;
  a.mask = B.mask;
  a.nchild = B.nchild;
  a.cfc = B.cfc;
  a.cslot = B.cslot;
  a.spos = B.spos;
  a.smass = B.smass;
  a.nodes = B.nodes;
  a.msum = B.msum;
  a.qmom = B.qmom;
  a.qpack = B.qpack;
  a.meta = B.meta;
  a.info = B.info;
  a.tiles = B.tiles;
  a.subs = B.subs;
  a.pieces = B.pieces;
  a.tops = B.tops;
  a.highs = B.highs;
  a.highs2 = B.highs2;
  a.by_level = reinterpret_cast<int32_t *>(B.vals[0]);  // (the sort is done with both)
  a.level_count = reinterpret_cast<int32_t *>(B.hist);
  // The scan: one workgroup alone for up to 16384 particles; tiles of 16384
  // again where tiles of 4096 would be more than 4096.
  if (B.n <= 16 * 1024 || B.n > ((int64_t)1 << 24)) {
    const unsigned nt = (unsigned)((B.n + 16 * 1024 - 1) / (16 * 1024));
    if (nt > 1) k_child_sums<1024><<<nt, 1024, 0, s>>>(a);
    k_child_scan<1024><<<nt, 1024, 0, s>>>(a);
  } else {
    const unsigned nt = (unsigned)((B.n + 16 * 256 - 1) / (16 * 256));
    k_child_sums<256><<<nt, 256, 0, s>>>(a);
    k_child_scan<256><<<nt, 256, 0, s>>>(a);
  }
  if (B.any_empty) empty_roots_device(B, s);
  if (quad_subtrees(B.n, B.qmom != nullptr))
    launch<kSubQuad, true>(a, s);
  else if (subtree_particles(B.n, B.qmom != nullptr, B.largest) == kSubFew)
    launch<kSubFew, false>(a, s);
  else
    launch<kSub, false>(a, s);
  if (B.qmom && !quad_subtrees(B.n, true)) second_moments(a, s);
}

}  // namespace bh
