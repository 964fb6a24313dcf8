// Force sum over the interaction lists (Eq. 1, FP32 with group-relative
// coordinates, partial sums folded into FP64).
//
// Work items are (group, block of 64 members, or the group's remainder); a
// persistent grid of single-wave workgroups pulls items from eight atomic
// queues, one per XCD, which hold the items of each group next to each other
// (so that the blocks of a group read its list through the same L2).
// A block of m members uses R lane partitions of W = 64/R >= m lanes, one
// member per lane;
// partition `part` takes list entries part, part + R, ...  With R = 1 every
// lane reads the same entry, so entries are fetched with scalar loads and used
// as scalar operands.  Per term a lane computes dx = x_j - x_i (near entries:
// from the FP32 value and its rounding residue), r^2 = |dx|^2 + eps^2 (FMA),
// v_rsq_f32, and accumulates m r^-3 dx and m r^-1, the terms of a block of
// entries written stage by stage so that dependent instructions issue far
// apart.  After each list chunk the FP32 partial sums are folded into FP64.  A
// member's own entry is in the near list with dx = 0 exactly: it adds 0 force
// and m_i/eps potential, removed at the end.
//
// Quadrupole sums (a template variant): a cell entry also adds the
// second-order term of the softened potential of its particles about their
// centre of mass, from the cell's second moments S (FP32, packed as 3 S and
// the trace, read by node slot: far entries carry the slot in a parallel
// array, near entries in the .w of their residue).  With u = dx, R^-1 as above and T = tr S:
//   potential  -3 (u.S.u) / (2 R^5) + T / (2 R^3)
//   force      -3 S u / R^5 + (15 (u.S.u) / (2 R^7) - 3 T / (2 R^5)) u.
#include "bh_device.h"
#include "force_terms.h"

namespace bh {

namespace {

// U entries against this lane's member; with QUAD, sl[u] is the node slot of a
// far entry (near entries: l[u].w), -1 for a particle.  The moments are
// fetched first (a particle's slot is clamped to 0 and its values unused), so
// that the monopole terms hide their latency.
template <int U, bool NEAR, bool QUAD = false>
__device__ __forceinline__ void terms(Member &M, const float4 (&e)[U], const float4 (&l)[U], float eps2,
                                      const int (&sl)[U], const float4 *__restrict__ qpack) {
  float4 qa[U], qb[U];
  bool cell[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int slot = QUAD ? (NEAR ? __float_as_int(l[u].w) : sl[u]) : -1;
    cell[u] = slot >= 0;
    if (QUAD) {
      const int64_t at = 2 * (int64_t)max(slot, 0);
      qa[u] = qpack[at];
      qb[u] = qpack[at + 1];
    }
  }
  entry_terms<U, NEAR, QUAD>(M, e, l, eps2, cell, qa, qb);
}

constexpr int kU = 8;      // entries per block of terms
constexpr int kUQuad = 4;  // the same for the quadrupole sums (register pressure)

// One chunk with R lane partitions: partition `part` takes entries part,
// part + R, ...; R is a compile-time constant so that the four entries of a
// block are loaded at constant offsets from one running pointer.  hs: the
// node slots of far entries (QUAD only).
template <bool NEAR, int R, bool QUAD>
__device__ __forceinline__ void chunk_part(Member &M, const float4 *__restrict__ h, const float4 *__restrict__ l,
                                           const int *__restrict__ hs, const float4 *__restrict__ qpack, int n,
                                           int part, float eps2) {
  constexpr int B = QUAD ? 2 : 4;  // entries per block (register pressure of the quadrupole terms)
  const int mine = (n - part + R - 1) / R;
  const float4 *ph = h + part;
  const float4 *pl = l + part;
  const int *ps = QUAD && !NEAR ? hs + part : nullptr;
  int t = 0;
  for (; t + B <= mine; t += B, ph += B * R, pl += B * R) {
    float4 e4[B], r4[B];
    int s4[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      e4[u] = ph[u * R];
      r4[u] = NEAR ? pl[u * R] : e4[u];
      s4[u] = (QUAD && !NEAR) ? ps[u * R] : -1;
    }
    if (QUAD && !NEAR) ps += B * R;
    terms<B, NEAR, QUAD>(M, e4, r4, eps2, s4, qpack);
  }
  for (; t < mine; ++t, ph += R, pl += R) {
    const float4 e1[1] = {ph[0]}, r1[1] = {NEAR ? pl[0] : ph[0]};
    int s1[1] = {-1};
    if (QUAD && !NEAR) {
      s1[0] = ps[0];
      ps += R;
    }
    terms<1, NEAR, QUAD>(M, e1, r1, eps2, s1, qpack);
  }
}

// n entries of one chunk: values at h[0..n), residues at l[0..n) when NEAR,
// node slots at hs[0..n) for far entries with QUAD.
template <bool NEAR, bool QUAD = false>
__device__ __forceinline__ void chunk_sum(Member &M, const float4 *__restrict__ h, const float4 *__restrict__ l,
                                          int n, int R, int part, float eps2, const int *__restrict__ hs = nullptr,
                                          const float4 *__restrict__ qpack = nullptr) {
  constexpr bool FS = QUAD && !NEAR;  // far slots to load
  constexpr int KU = QUAD ? kUQuad : kU;  // entries per block
  float4 e[KU], r[KU];
  int sl[KU];
#pragma unroll
  for (int u = 0; u < KU; ++u) sl[u] = -1;
  if (R == 1) {
    // every lane takes the same entries: scalar loads, scalar operands; the
    // next block is fetched while the current one is summed
    int t = 0;
    if (n >= KU) {
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        e[u] = h[u];
        r[u] = NEAR ? l[u] : e[u];
        if (FS) sl[u] = hs[u];
      }
      for (t = KU; t + KU <= n; t += KU) {
        float4 ne[KU], nr[KU];
        int ns[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
          ne[u] = h[t + u];
          nr[u] = NEAR ? l[t + u] : ne[u];
          ns[u] = FS ? hs[t + u] : -1;
        }
        terms<KU, NEAR, QUAD>(M, e, r, eps2, sl, qpack);
#pragma unroll
        for (int u = 0; u < KU; ++u) {
          e[u] = ne[u];
          r[u] = nr[u];
          sl[u] = ns[u];
        }
      }
      terms<KU, NEAR, QUAD>(M, e, r, eps2, sl, qpack);
    }
    for (; t < n; ++t) {
      const float4 e1[1] = {h[t]}, r1[1] = {NEAR ? l[t] : h[t]};
      const int s1[1] = {FS ? hs[t] : -1};
      terms<1, NEAR, QUAD>(M, e1, r1, eps2, s1, qpack);
    }
  } else {
    switch (R) {
      case 2: chunk_part<NEAR, 2, QUAD>(M, h, l, hs, qpack, n, part, eps2); break;
      case 4: chunk_part<NEAR, 4, QUAD>(M, h, l, hs, qpack, n, part, eps2); break;
      case 8: chunk_part<NEAR, 8, QUAD>(M, h, l, hs, qpack, n, part, eps2); break;
      case 16: chunk_part<NEAR, 16, QUAD>(M, h, l, hs, qpack, n, part, eps2); break;
      case 32: chunk_part<NEAR, 32, QUAD>(M, h, l, hs, qpack, n, part, eps2); break;
      default: chunk_part<NEAR, 64, QUAD>(M, h, l, hs, qpack, n, part, eps2); break;
    }
  }
  fold(M);
}

// The list data is read-only here; as separate restrict arguments the
// compiler can fetch wave-uniform entries with scalar loads.  QUAD: the
// quadrupole variant (far_slot and qpack set).
template <bool QUAD>
__global__ __launch_bounds__(kWave) void k_force_lists(ForceArgs a, const float4 *__restrict__ far_pool,
                                                       const int32_t *__restrict__ far_next,
                                                       const float4 *__restrict__ near_pool,
                                                       const int32_t *__restrict__ near_next,
                                                       const int32_t *__restrict__ glists,
                                                       const int32_t *__restrict__ items,
                                                       const int32_t *__restrict__ far_slot,
                                                       const float4 *__restrict__ qpack) {
  const int lane = lane_id();
  // workgroups are dealt to the XCDs round robin: this wave's XCD queue
  // first, then the others
  const int xcd = blockIdx.x & 7;
  int tried = 0;
  for (;;) {
    int it = -1;
    while (tried < 8) {
      // (a provably uniform queue index keeps the take a single atomic)
      const int x = __builtin_amdgcn_readfirstlane((xcd + tried) & 7);
      const int s0 = a.xstart[x], s1 = a.xstart[x + 1];
      const int q = take_one(&a.info->fq[x * kLineInts], lane);
      if (s0 + q < s1) {
        it = s0 + q;
        break;
      }
      ++tried;
    }
    if (it < 0) break;
    const int g = items[2 * it], iv = items[2 * it + 1];
    const int blk = iv & 255, segl = iv >> 8;
    const int gf = a.ginfo[3 * g], gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    int fh, fn, nh, nn, prow = -1;
    if (segl == 0) {
      fh = glists[4 * g];
      fn = glists[4 * g + 1];
      nh = glists[4 * g + 2];
      nn = glists[4 * g + 3];
    } else {
      // one segment of a split group: partial sums go to its rows
      const int p = a.gsegfirst[g] + segl - 1;
      const Segment sg = a.segs[a.seg_order[p]];
      fh = sg.fh;
      fn = sg.fn;
      nh = sg.nh;
      nn = sg.nn;
      prow = a.pbase[p];
    }
    if ((fn > 0 && fh < 0) || (nn > 0 && nh < 0)) continue;  // incomplete list (reported by the walk)
    // members [b0, b1) of the group: full blocks of 64, then the remainder,
    // which takes several lane partitions when it is small
    const int b0 = blk * kWave, b1 = min(gc, b0 + kWave);
    const int m = b1 - b0;
    int R = 1;
    while (R < kWave && m * (2 * R) <= kWave) R *= 2;
    const int W = kWave / R;
    const int part = lane / W, u = lane % W;

    double cen[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      cen[k] = __dmul_rn(__dadd_rn(a.gbox[6 * (int64_t)g + k], a.gbox[6 * (int64_t)g + 3 + k]), 0.5);
    const double eps = a.par[gs].eps;
    const float eps2 = (float)(eps * eps);

    Member M;
    {
      double rx = 0.0, ry = 0.0, rz = 0.0;
      if (u < m) {
        const double *q = a.spos + 3 * (int64_t)(gf + b0 + u);
        rx = __dsub_rn(q[0], cen[0]);
        ry = __dsub_rn(q[1], cen[1]);
        rz = __dsub_rn(q[2], cen[2]);
      }
      member_init(M, rx, ry, rz);
    }

    int ch = fh;
    for (int left = fn; left > 0;) {
      const int n = min(left, a.far_tile);
      const float4 *base = far_pool + (int64_t)ch * a.far_tile;
      chunk_sum<false, QUAD>(M, base, base, n, R, part, eps2, QUAD ? far_slot + (int64_t)ch * a.far_tile : nullptr,
                             qpack);
      left -= n;
      if (left > 0) ch = far_next[ch];
    }
    ch = nh;
    for (int left = nn; left > 0;) {
      const int n = min(left, a.near_tile);
      const float4 *base = near_pool + (int64_t)ch * (2 * a.near_tile);
      chunk_sum<true, QUAD>(M, base, base + a.near_tile, n, R, part, eps2, nullptr, qpack);
      left -= n;
      if (left > 0) ch = near_next[ch];
    }

    // reduce partitions, remove the self term, write in input order
    double vx = M.dx, vy = M.dy, vz = M.dz, vp = M.dp;
    for (int b = W; b < kWave; b <<= 1) {
      vx += shfl_xor_d(vx, b);
      vy += shfl_xor_d(vy, b);
      vz += shfl_xor_d(vz, b);
      vp += shfl_xor_d(vp, b);
    }
    if (prow >= 0) {
      if (part == 0 && u < m) {
        double *q = a.psum + 4 * ((int64_t)prow + b0 + u);
        q[0] = vx;
        q[1] = vy;
        q[2] = vz;
        q[3] = vp;
      }
    } else if (part == 0 && u < m) {
      const int i = gf + b0 + u;
      const double self = self_potential(a.smass[i], eps2);
      const int o = a.perm[i];
      a.acc[3 * (int64_t)o] = (float)vx;
      a.acc[3 * (int64_t)o + 1] = (float)vy;
      a.acc[3 * (int64_t)o + 2] = (float)vz;
      a.pot[o] = (float)(self - vp);
    }
  }
}

// Rows of the tile sums: one per tile of each group's list (far tiles, then
// near ones), numbered by groups; list statistics.  One workgroup; bound by
// following the tiles' links (a dozen reads).  Rows beyond the room for them are
// counted and not written.
__global__ __launch_bounds__(1024) void k_tile_rows(TileArgs a) {
  __shared__ int wsum[1024 / kWave];
  const int t = threadIdx.x, w = t / kWave;
  if (a.info->err & (kErrPool | kErrWide)) {  // lists incomplete: the host walks again
    if (t == 0) a.info->tile_rows = a.info->tile_need = 0;
    return;
  }
  const int G = a.info->n_groups;
  int base = 0, longest = 0;
  unsigned long long inter = 0, entries = 0;
  for (int g0 = 0; g0 < G; g0 += 1024) {
    const int g = g0 + t;
    int4 L = make_int4(-1, 0, -1, 0);
    if (g < G) {
      L = reinterpret_cast<const int4 *>(a.glists)[g];
      const int len = max(a.glist[g], 0);
      inter += (unsigned long long)a.ginfo[3 * g + 1] * (unsigned long long)max(len - 1, 0);
      entries += (unsigned long long)len;
      longest = max(longest, len);
    }
    const int nf = (L.y + a.far_tile - 1) / a.far_tile, rows = nf + (L.w + a.near_tile - 1) / a.near_tile;
    const int inc = wave_inclusive_sum(rows);
    if (lane_id() == kWave - 1) wsum[w] = inc;
    __syncthreads();
    int row = base + inc - rows;
    for (int k = 0; k < 1024 / kWave; ++k) {
      if (k < w) row += wsum[k];
      base += wsum[k];
    }
    __syncthreads();
    if (g < G) a.gblocks[g] = make_int2(row, rows);
    int ch = L.x;
    for (int left = L.y; left > 0 && row < a.row_cap; left -= a.far_tile) {
      a.tinfo[row++] = make_int4(g, ch, min(left, a.far_tile), 0);
      if (left > a.far_tile) ch = a.far_next[ch];
    }
    ch = L.z;
    for (int left = L.w; left > 0 && row < a.row_cap; left -= a.near_tile) {
      a.tinfo[row++] = make_int4(g, ch, min(left, a.near_tile), 1);
      if (left > a.near_tile) ch = a.near_next[ch];
    }
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    inter += __shfl_xor(inter, d, kWave);
    entries += __shfl_xor(entries, d, kWave);
    longest = max(longest, __shfl_xor(longest, d, kWave));
  }
  if (lane_id() == 0 && entries) {
    atomicAdd(&a.info->interactions, inter);
    atomicAdd(&a.info->list_entries, entries);
    atomicMax(&a.info->max_list, longest);
  }
  if (t == 0) {
    const bool fits = base <= a.row_cap;
    if (!fits) atomicOr(&a.info->err, kErrPool);  // (the sums leave at once, the host makes room)
    a.info->tile_rows = fits ? base : 0;
    a.info->tile_need = base;
  }
}

// The sums of k_force_lists taken apart by tiles: a workgroup per tile, a wave
// per block of 64 members, each member's FP32 chain over the tile's entries
// (or its lane partition's) the same as there, so the values differ only in
// the order in which tiles and partitions are added in FP64.  For too few
// groups to fill the chip with a wave each: the longest list no longer decides
// (30,011 Plummer particles: 602 us with a wave per group, 86 with a workgroup
// per tile; 100,003 in a sphere 151, with 16 rather than 8 KiB of LDS and 4
// rather than 8 entries at a time 188).  Entries are staged in LDS: a lone wave
// waits for every scalar load.
template <bool QUAD>
__global__ __launch_bounds__(256) void k_force_tiles(TileArgs a) {
  constexpr int kStage = QUAD ? 256 : 512;
  __shared__ float4 e[kStage + (QUAD ? kStage : 0)];  // entries; the second half (QUAD: array) residues
  __shared__ float4 qs[QUAD ? 2 * kStage : 1];
  __shared__ int32_t sl[QUAD ? kStage : 1];
  constexpr int kHalf = QUAD ? kStage : kStage / 2;
  const int t = threadIdx.x, NT = blockDim.x, lane = lane_id(), blk = t / kWave;
  const int rows = a.info->tile_rows;
  for (int row = blockIdx.x; row < rows; row += gridDim.x) {
    const int4 b = a.tinfo[row];
    const int g = __builtin_amdgcn_readfirstlane(b.x), cnt = __builtin_amdgcn_readfirstlane(b.z);
    const bool near = __builtin_amdgcn_readfirstlane(b.w) != 0;
    const int ch = __builtin_amdgcn_readfirstlane(b.y);
    const float4 *pool = near ? a.near_pool + (int64_t)ch * (2 * a.near_tile) : a.far_pool + (int64_t)ch * a.far_tile;
    const int gf = a.ginfo[3 * g], gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    const int m = min(gc - blk * kWave, kWave);  // (may be <= 0)
    int R = 1;
    while (R < kWave && max(m, 1) * (2 * R) <= kWave) R *= 2;
    const int W = kWave / R, part = lane / W, u = lane % W;
    double cen[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      cen[k] = __dmul_rn(__dadd_rn(a.gbox[6 * (int64_t)g + k], a.gbox[6 * (int64_t)g + 3 + k]), 0.5);
    const double eps = a.par[gs].eps;
    const float eps2 = (float)(eps * eps);
    Member M;
    {
      double x = 0.0, y = 0.0, z = 0.0;
      if (u < m) {
        const double *q = a.spos + 3 * (int64_t)(gf + blk * kWave + u);
        x = __dsub_rn(q[0], cen[0]);
        y = __dsub_rn(q[1], cen[1]);
        z = __dsub_rn(q[2], cen[2]);
      }
      member_init(M, x, y, z);
    }
    const int step = near && !QUAD ? kHalf : kStage;
    for (int s0 = 0; s0 < cnt; s0 += step) {
      const int s = min(step, cnt - s0);
      __syncthreads();
      for (int k = t; k < s; k += NT) {
        e[k] = pool[s0 + k];
        int slot = -1;
        if (near) {
          const float4 r = pool[a.near_tile + s0 + k];
          e[kHalf + k] = r;
          if (QUAD) slot = __float_as_int(r.w);
        } else if (QUAD) {
          slot = a.far_slot[(int64_t)ch * a.far_tile + s0 + k];
        }
        if (QUAD) {
          sl[k] = slot;
          const int64_t q = 2 * (int64_t)max(slot, 0);
          qs[2 * k] = a.qpack[q];
          qs[2 * k + 1] = a.qpack[q + 1];
        }
      }
      __syncthreads();
      // (with second moments in the same blocks as chunk_sum and chunk_part)
      if (m > 0) {
        if (QUAD && R == 1) {
          if (near)
            stage_sum<true, QUAD, kUQuad>(M, e, e + kHalf, sl, qs, 0, s, part, R, eps2);
          else
            stage_sum<false, QUAD, kUQuad>(M, e, e, sl, qs, 0, s, part, R, eps2);
        } else if (near) {
          stage_sum<true, QUAD, QUAD ? 2 : kU>(M, e, e + kHalf, sl, qs, 0, s, part, R, eps2);
        } else {
          stage_sum<false, QUAD, QUAD ? 2 : kU>(M, e, e, sl, qs, 0, s, part, R, eps2);
        }
      }
    }
    fold(M);
    double v[4] = {M.dx, M.dy, M.dz, M.dp};
    for (int d = W; d < kWave; d <<= 1)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += shfl_xor_d(v[k], d);
    if (part == 0 && u < m) {
      double2 *q = reinterpret_cast<double2 *>(a.psum + 4 * ((int64_t)row * a.n_crit + blk * kWave + u));
      q[0] = make_double2(v[0], v[1]);
      q[1] = make_double2(v[2], v[3]);
    }
  }
}

}  // namespace

void tile_rows_device(const TileArgs &a, hipStream_t s) { k_tile_rows<<<1, 1024, 0, s>>>(a); }

void force_tiles_device(const TileArgs &a, int num_cu, hipStream_t s) {
  const int nt = a.n_crit <= 64 ? 64 : (a.n_crit <= 128 ? 128 : 256);
  if (a.far_slot && a.qpack)
    k_force_tiles<true><<<(unsigned)(num_cu * 8), nt, 0, s>>>(a);
  else
    k_force_tiles<false><<<(unsigned)(num_cu * 16), nt, 0, s>>>(a);
}

int force_lists_blocks_per_cu(bool quad) {
  int b = 0;
  const hipError_t e = quad ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_force_lists<true>, kWave, 0)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_force_lists<false>, kWave, 0);
  if (e != hipSuccess || b < 1) b = 8;
  return b;
}

void force_lists_device(const ForceArgs &a, int grid, hipStream_t s) {
  if (a.far_slot && a.qpack)
    k_force_lists<true><<<(unsigned)grid, kWave, 0, s>>>(a, a.far_pool, a.far_next, a.near_pool, a.near_next,
                                                         a.glists, a.items, a.far_slot, a.qpack);
  else
    k_force_lists<false><<<(unsigned)grid, kWave, 0, s>>>(a, a.far_pool, a.far_next, a.near_pool, a.near_next,
                                                          a.glists, a.items, nullptr, nullptr);
}

}  // namespace bh
