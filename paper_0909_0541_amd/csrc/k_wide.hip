// Force call with quadrupoles for sizes that leave the chip idle with one wave
// per group: the group walk by a whole workgroup, and the list summed in equal
// blocks by many workgroups; and outliers at every size, with or without
// quadrupoles.
//
// With a few hundred or thousand groups, the single-wave walk and sum
// (k_walk_lists, k_force_lists) run as long as their longest chain: a wave
// takes about a microsecond per batch of 64 nodes and, alone on its SIMD, up
// to 0.1 us per list entry, and one group with a sparse box (the outskirts of
// a Plummer sphere) opens the whole tree.  Here
//   k_walk_wide     one workgroup of NT threads per group tests up to NT
//                   nodes per iteration (the same opening test and the same
//                   far/near rule, so the same lists as sets) and writes the
//                   list in blocks of BL far or BL/2 near entries taken from
//                   one pool;
//   k_force_blocks  one workgroup per block sums its entries for the group's
//                   members and writes a row of FP64 partial sums;
//   k_block_reduce  adds each member's rows in list order, removes the self
//                   term and writes the outputs.
// Work is even whatever the lists' lengths, and a member's sums are FP32 over
// at most 256 entries at a time, then FP64 in an order fixed by the walk, so
// the results do not depend on scheduling.
//
// Outliers.  A few groups with sparse boxes (1 to 6 of a Plummer sphere's
// thousands) have lists of nearly every particle, hundreds of times the
// median, and one workgroup (or, on larger trees, one wave of k_walk_lists)
// would hold the launch open for them.  A walk that has tested outlier_cap
// nodes gives its group up to this path: the group is walked again from the
// root over its large cells only, the subtrees below them that have to be
// opened become tasks of kTaskNodes nodes each, and a second launch walks the
// tasks, one workgroup each.  A task's rows follow the group's own in task
// order, so the sums are fixed here too (k_task_reduce).
#include <algorithm>

#include "bh_device.h"
#include "force_terms.h"

namespace bh {

namespace {

constexpr int kWideReserve = 8 * 24;         // growth bound in one-node mode
constexpr int kWideIds = 3 * 1024 + 64;      // block ids of one list (BL >= n / 1024: at most 3 n / BL + 2)
constexpr int kStage = 256;                  // entries staged in LDS at a time by the sum

// One workgroup per unit: a group, an outlier group over its large cells
// (top), or a task (below).  The stack holds single nodes; an iteration takes
// up to NT from the top (as many as leave room for eight children each, at
// least one: then the walk is depth first and grows the stack by at most 7 a
// level).  The children of a bucket (coincident particles, any number) are
// particles and are taken straight as a range.  Entries go to places given
// by block-wide ranks (wave by wave, lane by lane), so the list order is
// fixed.  Bound by the chain of an iteration: one round of node reads from
// L2 or beyond and two barriers, about 2 us, so NT is as large as leaves every
// compute unit a group (8192-particle Plummer sphere, 195 groups: 129 us at
// 256 threads, 77 at 512, 63 at 1024; 100,003 particles in 1088 groups: 96 us
// at 256, 92 at 512).  Device-wide atomics on one line queue up at some 50 ns
// each, so a unit makes one (its rows) and one per kSpare blocks, asked for
// ahead; with seven per group the same 1088 groups took 96 us, now 75, and
// 1280 workgroups asking for blocks without a unit to walk took 70 us.
constexpr int kUnitGroups = 0, kUnitOutliers = 1, kUnitTasks = 2;

template <int NT, bool SLOTS, int MODE>
__global__ __launch_bounds__(NT) void k_walk_wide(WideArgs a) {
  constexpr int NW = NT / kWave;
  constexpr int kWideStack = 16 * NT;
  __shared__ int32_t stk[kWideStack];
  __shared__ int32_t ids[kWideIds];  // far blocks from the front, near blocks from the back
  __shared__ int2 big[NT];
  __shared__ int4 wt[NW];
  __shared__ double wm[NW];
  __shared__ int sh_g, sh_id;
  const int t = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(t / kWave);
  const int G = a.info->n_groups;
  const int nslots = a.nsys + a.info->n_slots;
  const int BL = a.block, BN = a.block / 2, bl = a.block_log;
  // blocks in hand: [spare, spare_end), taken from the pool kSpare at a time;
  // the next run is asked for while the current one still lasts
  int spare = 0, spare_end = 0;
  int run = 0;  // (thread 0) the run asked for
  int *queue = MODE == kUnitTasks ? &a.info->queue2 : &a.info->queue;
  const int units = MODE == kUnitGroups     ? G
                    : MODE == kUnitOutliers ? min(a.info->n_out - a.out_first, a.lot)
                                            : min(a.info->tasks, a.lot * kOutTasks);
  if (MODE == kUnitOutliers && a.out_limit > 0 && a.info->n_out > a.out_limit && blockIdx.x == 0 && t == 0)
    atomicOr(&a.info->err, kErrWide);
  int unit = blockIdx.x;  // the first unit by place, the next ones from the queue
  if (unit < units && t == 0) run = atomicAdd(&a.info->blocks, kSpare);
  while (unit < units) {
    int unext = units;
    if (t == 0 && gridDim.x < units) unext = atomicAdd(queue, 1);  // (read at the end of this unit)
    int g = unit, oidx = unit;
    int4 task = make_int4(0, 0, 0, 0);
    if (MODE == kUnitOutliers) g = a.out[a.out_first + unit];
    if (MODE == kUnitTasks) {
      task = a.tasks[unit];
      g = task.x;
    }
    g = __builtin_amdgcn_readfirstlane(g);
    if (g < 0 || g >= G) {  // corrupt: report and leave
      if (t == 0) atomicOr(&a.info->err, kErrStack);
      break;
    }
    const int gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    double blo[3], bhi[3], cen[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      blo[k] = a.gbox[6 * (int64_t)g + k];
      bhi[k] = a.gbox[6 * (int64_t)g + 3 + k];
      cen[k] = __dmul_rn(__dadd_rn(blo[k], bhi[k]), 0.5);
    }
    double theta = a.theta_group ? (double)a.theta_group[g] : a.par[gs].theta;
    if (isnan(theta)) {
      theta = a.par[gs].theta;
      if (t == 0 && MODE == kUnitGroups) atomicAdd(&a.info->theta_fallback, 1);
    }
    if (!(theta >= 0.0 && theta <= 1.0)) {
      if (t == 0) atomicOr(&a.info->err, kErrTheta);
      theta = (theta > 1.0) ? 1.0 : 0.0;
    }
    const double side = a.sys[gs].side;
    const double side_theta = side / theta;  // l / theta = (side / theta) 2^-level exactly
    const int side_exp = ilogb(side);
    double hd2 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double e = __dsub_rn(bhi[k], blo[k]);
      hd2 = __dadd_rn(hd2, __dmul_rn(e, e));
    }
    const double near2 = __dmul_rn(hd2, 0.25 * kNearFrac * kNearFrac);

    bool top = MODE == kUnitOutliers;
    const int small = max(a.sys[gs].count >> 11, 64);  // cells of at most this many particles become tasks
    int cap = MODE == kUnitGroups ? outlier_cap(a.out_min, a.out_tree, a.n_crit, a.sys[gs].count, theta) : 0;
    int tcount = 0;  // task nodes
    int sp = 1, nbig = 0;
    int fcount = 0, ncount = 0, fblocks = 0, nblocks = 0;
    int visits = 0, budget = 4 * nslots + 4;
    bool ok = true, corrupt = false, too_long = false;
    double lmass = 0.0;
    if (MODE == kUnitTasks) {
      sp = min(max(task.z, 0), kTaskNodes);
      if (t < sp) stk[sp - 1 - t] = a.tnodes[task.y + t];
    } else if (t == 0) {
      stk[0] = gs;
    }
    __syncthreads();
    while (sp > 0 || nbig > 0) {
      if (--budget < 0) {
        corrupt = true;
        break;
      }
      int take, node = -1;
      int2 rng = make_int2(0, 0);
      const bool from_range = nbig > 0;
      if (from_range) {
        rng = big[nbig - 1];
        take = min(NT, rng.y);
        if (t < take) node = rng.x + t;
      } else {
        take = min(min(sp, NT), max(1, (kWideStack - kWideReserve - sp) / 7));
        if (t < take) node = stk[sp - 1 - t];
      }
      bool emit = false, near = false, bad = false, sub = false;
      const bool subs = MODE != kUnitTasks && top && tcount + NT <= kOutNodes;
      int nc = 0, child = 0;
      float4 hi4 = make_float4(0.f, 0.f, 0.f, 0.f), lo4 = hi4;
      if (t < take) {
        bad = node < 0 || node >= nslots;
        const NodeRec r = a.nodes[bad ? 0 : node];
        double d2 = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double below = __dsub_rn(blo[k], r.com[k]);
          const double above = __dsub_rn(r.com[k], bhi[k]);
          const double ek = fmax(0.0, fmax(below, above));
          d2 = (k == 0) ? __dmul_rn(ek, ek) : __dadd_rn(d2, __dmul_rn(ek, ek));
        }
        if (r.child < 0) {
          emit = true;  // a particle
        } else {
          // Eq. (2)/(3): far enough iff d^2 > (l/theta + s)^2
          double q = isfinite(r.l) ? ldexp(side_theta, ilogb(r.l) - side_exp) : r.l;
          q = __dadd_rn(q, r.s);
          emit = d2 > __dmul_rn(q, q);
          if (!emit && subs && r.count <= small) {
            sub = true;
          } else if (!emit) {
            nc = r.nchild;
            child = r.child;
          }
        }
        if (bad || (from_range && !emit)) {
          emit = sub = false;
          nc = 0;
          bad = true;
        }
        if (emit) {
          const double rx = __dsub_rn(r.com[0], cen[0]), ry = __dsub_rn(r.com[1], cen[1]),
                       rz = __dsub_rn(r.com[2], cen[2]);
          hi4 = make_float4((float)rx, (float)ry, (float)rz, (float)r.m);
          near = d2 <= near2;
          if (near)
            lo4 = make_float4((float)__dsub_rn(rx, (double)hi4.x), (float)__dsub_rn(ry, (double)hi4.y),
                              (float)__dsub_rn(rz, (double)hi4.z), __int_as_float(r.child < 0 ? -1 : node));
          lmass += r.m;
        }
        if (SLOTS) child = emit ? (r.child < 0 ? -1 : node) : child;
      }
      const bool wide = nc > 8;
      const unsigned long long fm = __ballot(emit && !near), nm = __ballot(near), bm = __ballot(wide),
                               badm = __ballot(bad), sm = __ballot(sub);
      const int pinc = wave_inclusive_sum(wide ? 0 : nc);
      // totals and this wave's offsets: two packed counts per word, the
      // waves' words scanned by every wave (far | near << 16 and
      // pushes | buckets << 16, a corrupt batch in the top bits)
      if (lane == kWave - 1)
        wt[wv] = make_int4(__popcll(fm) | (__popcll(nm) << 16),
                           pinc | (__popcll(bm) << 16) | (badm ? 1 << 27 : 0), __popcll(sm), 0);
      __syncthreads();
      const int4 mine = wt[lane & (NW - 1)];
      const int ei = wave_row_sum(mine.x), pi = wave_row_sum(mine.y);  // inclusive over the waves
      const int et = __builtin_amdgcn_readlane(ei, NW - 1), ptot = __builtin_amdgcn_readlane(pi, NW - 1);
      const int eo = wv ? __builtin_amdgcn_readlane(ei, wv - 1) : 0, pof = wv ? __builtin_amdgcn_readlane(pi, wv - 1) : 0;
      const int fo = eo & 0xffff, no = eo >> 16, po = pof & 0xffff, bo = pof >> 16;
      const int ft = et & 0xffff, nt = et >> 16, pt = ptot & 0xffff, bt = (ptot >> 16) & 0x7ff;
      corrupt = ((uint32_t)ptot >> 27) != 0;
      if (corrupt) break;  // the same on every thread
      visits += take;
      if (subs) {
        const int si = wave_row_sum(mine.z);
        const int so = wv ? __builtin_amdgcn_readlane(si, wv - 1) : 0;
        if (sub) a.tnodes[oidx * kOutNodes + tcount + so + rank_below(sm)] = node;
        tcount += __builtin_amdgcn_readlane(si, NW - 1);
      }
      // blocks for the entries to come
      const int kf = ((fcount + ft + BL - 1) >> bl) - fblocks, kn = ((ncount + nt + BN - 1) >> (bl - 1)) - nblocks;
      if (kf > 0 || kn > 0) {
        if (fblocks + kf + nblocks + kn > kWideIds) {  // (never where blocks hold n / 1024 entries)
          corrupt = too_long = true;
          break;
        }
        for (int k = 0; k < kf + kn; ++k) {
          if (spare == spare_end) {
            if (t == 0) {
              sh_id = run;
              run = atomicAdd(&a.info->blocks, kSpare);
            }
            __syncthreads();
            spare = __builtin_amdgcn_readfirstlane(sh_id);
            spare_end = spare + kSpare;
            __syncthreads();
          }
          if (spare >= a.block_cap) ok = false;  // keeps counting: the host grows the pool and walks again
          if (t == 0) ids[k < kf ? fblocks + k : kWideIds - 1 - nblocks - (k - kf)] = spare;
          ++spare;
        }
        fblocks += kf;
        nblocks += kn;
        __syncthreads();
      }
      if (ok && emit) {
        if (!near) {
          const int pos = fcount + fo + rank_below(fm);
          const int64_t at = (int64_t)ids[pos >> bl] * BL + (pos & (BL - 1));
          a.pool[at] = hi4;
          if (SLOTS) a.slot[at] = child;
        } else {
          const int pos = ncount + no + rank_below(nm);
          float4 *base = a.pool + (int64_t)ids[kWideIds - 1 - (pos >> (bl - 1))] * BL + (pos & (BN - 1));
          base[0] = hi4;
          base[BN] = lo4;
        }
      }
      fcount += ft;
      ncount += nt;
      // children onto the stack (the places taken have been read before the barrier)
      const int base = from_range ? sp : sp - take;
      if (nc > 0 && !wide) {
        int q = base + po + pinc - nc;
        for (int k = 0; k < nc; ++k) stk[q + k] = child + k;
      }
      if (from_range) {
        if (t == 0 && rng.y > take) big[nbig - 1] = make_int2(rng.x + take, rng.y - take);
        if (rng.y <= take) --nbig;
      } else if (bt > 0) {
        if (wide) big[bo + rank_below(bm)] = make_int2(child, nc);
        nbig = bt;
      }
      sp = base + pt;
      __syncthreads();
      if (cap > 0 && visits >= cap) {
        // an outlier: start again over the large cells
        cap = 0;
        if (t == 0) {
          const int o = take_outlier(a.info, a.lot);
          if (o >= 0) a.out[o] = g;
          sh_id = o;
        }
        __syncthreads();
        oidx = __builtin_amdgcn_readfirstlane(sh_id);
        if (oidx >= 0) {
          top = true;
          sp = 1;
          nbig = fcount = ncount = fblocks = nblocks = 0;
          lmass = 0.0;
          if (t == 0) stk[0] = gs;
        }
        __syncthreads();
      }
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) lmass += shfl_xor_d(lmass, d);
    if (lane == 0) wm[wv] = lmass;
    __syncthreads();
    // The list's blocks, far then near, get consecutive rows.  A list that did
    // not fit gets none: rows then number blocks of the pool, each once, and
    // never exceed its capacity, that of the arrays over rows.
    const int nused = corrupt || !ok ? 0 : fblocks + nblocks;
    if (t == 0) {
      double m = wm[0];
      for (int w = 1; w < NW; ++w) m += wm[w];
      const int len = corrupt ? 0 : fcount + ncount;
      if (corrupt) atomicOr(&a.info->err, too_long ? kErrWide : kErrStack);
      if (!ok) atomicOr(&a.info->err, kErrPool);
      if (corrupt) m = 0.0;
      const int row = atomicAdd(&a.info->rows, nused);
      sh_id = row;
      if (MODE == kUnitTasks) {
        a.trows[unit] = make_int4(row, nused, len, visits);
        a.tnear[unit] = ncount;
        a.tmass[unit] = m;
      } else if (top) {
        // the outlier's own part; its tasks are consecutive
        const int nt = (tcount + kTaskNodes - 1) / kTaskNodes;
        const int t0 = atomicAdd(&a.info->tasks, nt);
        OutInfo o;
        o.g = g;
        o.task0 = t0;
        o.tasks = nt;
        o.row0 = row;
        o.rows = nused;
        o.len = len;
        o.visits = visits;
        o.near = ncount;
        o.mass = m;
        a.outinfo[oidx] = o;
        sh_g = t0;
        if (MODE == kUnitGroups) a.gblocks[g] = make_int2(0, -1);
      } else {
        a.glist[g] = len;
        a.gmass[g] = m;
        a.gblocks[g] = make_int2(row, nused);
        a.gstat[g] = make_int2(visits, ncount);
      }
    }
    __syncthreads();
    if (nused > 0) {
      const int row = __builtin_amdgcn_readfirstlane(sh_id);
      for (int k = t; k < nused; k += NT) {
        const bool nr = k >= fblocks;
        const int j = nr ? k - fblocks : k;
        const int id = ids[nr ? kWideIds - 1 - j : j];
        const int cnt = nr ? min(BN, ncount - j * BN) : min(BL, fcount - j * BL);
        a.binfo[row + k] = make_int4(g, id, cnt, nr ? 1 : 0);
      }
    }
    if (MODE != kUnitTasks && top) {
      const int t0 = __builtin_amdgcn_readfirstlane(sh_g);
      for (int k = t; k < (tcount + kTaskNodes - 1) / kTaskNodes; k += NT)
        if (t0 + k < a.lot * kOutTasks)
          a.tasks[t0 + k] = make_int4(g, oidx * kOutNodes + kTaskNodes * k, min(kTaskNodes, tcount - kTaskNodes * k), 0);
      __syncthreads();
    }
    if (t == 0) sh_g = unext;
    __syncthreads();
    unit = gridDim.x + __builtin_amdgcn_readfirstlane(sh_g);
    __syncthreads();
  }
}

// Statistics of the groups a workgroup's threads have seen, added to the
// counters wave by wave.
struct ListStats {
  unsigned long long inter = 0, entries = 0, visits = 0, near = 0;
  int longest = 0;
  __device__ __forceinline__ void add(int count, int len, int v, int nr) {
    inter += (unsigned long long)count * (unsigned long long)max(len - 1, 0);
    entries += (unsigned long long)len;
    visits += (unsigned long long)v;
    near += (unsigned long long)nr;
    longest = max(longest, len);
  }
  __device__ __forceinline__ void store(DevInfo *info) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      inter += __shfl_xor(inter, d, kWave);
      entries += __shfl_xor(entries, d, kWave);
      visits += __shfl_xor(visits, d, kWave);
      near += __shfl_xor(near, d, kWave);
      longest = max(longest, __shfl_xor(longest, d, kWave));
    }
    if (lane_id() == 0) {
      atomicAdd(&info->interactions, inter);
      atomicAdd(&info->list_entries, entries);
      atomicAdd(&info->node_visits, visits);
      atomicAdd(&info->near_entries, near);
      atomicMax(&info->max_list, longest);
    }
  }
};

// One workgroup of four waves per list block.  Groups of at most 64 members
// take the entries in four parts (one per wave), of at most 128 in two parts
// with a wave per member block, larger ones whole with a wave per member
// block; a block of m <= 32 members also uses 64/m lane partitions.  Entries
// are staged in LDS and read as broadcasts (a lone wave waits for every
// scalar load; LDS keeps up with four waves: 123 us against 166 for 100,003
// particles, 882 against 1498 with quadrupoles for 300,001).  Bound by FP32
// issue at 2.4e12 lane interactions per second.
template <bool QUAD>
__global__ __launch_bounds__(256) void k_force_blocks(WideArgs a) {
  __shared__ float4 e[kStage], l[kStage];
  __shared__ float4 qs[QUAD ? 2 * kStage : 1];
  __shared__ int32_t sl[QUAD ? kStage : 1];
  __shared__ double part[4][kWave][4];
  const int t = threadIdx.x, lane = lane_id(), wv = t / kWave;
  if (a.info->err & (kErrPool | kErrWide)) return;  // lists incomplete: the host walks again
  const int rows = a.info->rows;
  for (int row = blockIdx.x; row < rows; row += gridDim.x) {
    const int4 b = a.binfo[row];
    const int g = __builtin_amdgcn_readfirstlane(b.x), cnt = __builtin_amdgcn_readfirstlane(b.z);
    const bool near = __builtin_amdgcn_readfirstlane(b.w) != 0;
    const int64_t at = (int64_t)__builtin_amdgcn_readfirstlane(b.y) * a.block;
    const int gf = a.ginfo[3 * g], gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    const int mb = gc <= kWave ? 1 : (gc <= 2 * kWave ? 2 : 4);  // waves that differ by member block
    const int ep = 4 / mb;                                       // entry parts
    const int blk = wv % mb, ept = wv / mb;
    const int m = min(gc - blk * kWave, kWave);  // may be <= 0 (three member blocks)
    int R = 1;
    while (R < kWave && max(m, 1) * (2 * R) <= kWave) R *= 2;
    const int W = kWave / R, sub = lane / W, u = lane % W;
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
    for (int s0 = 0; s0 < cnt; s0 += kStage) {
      const int s = min(kStage, cnt - s0);
      const int lo = s * ept / ep, hi = s * (ept + 1) / ep;  // this wave's part
      __syncthreads();
      if (t < s) {
        e[t] = a.pool[at + s0 + t];
        int slot = -1;
        if (near) {
          l[t] = a.pool[at + a.block / 2 + s0 + t];
          if (QUAD) slot = __float_as_int(l[t].w);
        } else if (QUAD) {
          slot = a.slot[at + s0 + t];
        }
        if (QUAD) {
          sl[t] = slot;
          const int64_t k = 2 * (int64_t)max(slot, 0);
          qs[2 * t] = a.qpack[k];
          qs[2 * t + 1] = a.qpack[k + 1];
        }
      }
      __syncthreads();
      if (near)
        stage_sum<true, QUAD>(M, e, l, sl, qs, lo, hi, sub, R, eps2);
      else
        stage_sum<false, QUAD>(M, e, l, sl, qs, lo, hi, sub, R, eps2);
      fold(M);
    }
    double v[4] = {M.dx, M.dy, M.dz, M.dp};
    for (int d = W; d < kWave; d <<= 1)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += shfl_xor_d(v[k], d);
    if (ep > 1) {
#pragma unroll
      for (int k = 0; k < 4; ++k) part[wv][lane][k] = v[k];
      __syncthreads();
      if (ept == 0)
        for (int p = 1; p < ep; ++p)
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] += part[wv + p * mb][lane][k];
    }
    if (ept == 0 && sub == 0 && u < m) {
      double2 *q = reinterpret_cast<double2 *>(a.psum + 4 * ((int64_t)row * a.n_crit + blk * kWave + u));
      q[0] = make_double2(v[0], v[1]);
      q[1] = make_double2(v[2], v[3]);
    }
    __syncthreads();
  }
}

// One member per thread: its rows in list order (far blocks, then near ones),
// four loads in flight.  With STATS the last workgroup adds up the list
// statistics (an atomic per group and counter, all on one line, took longer
// than the walk).
template <bool STATS>
__global__ __launch_bounds__(256) void k_block_reduce(WideArgs a, int width) {
  if (a.info->err & (kErrPool | kErrWide)) return;
  const int G = a.info->n_groups;
  if (STATS && blockIdx.x == gridDim.x - 1) {
    ListStats st;
    for (int g = threadIdx.x; g < G; g += 256) {
      if (a.gblocks[g].y < 0) continue;  // (an outlier: k_task_reduce)
      const int2 v = a.gstat[g];
      st.add(a.ginfo[3 * g + 1], a.glist[g], v.x, v.y);
    }
    st.store(a.info);
    return;
  }
  const int per = 256 / width;  // groups per workgroup
  const int u = threadIdx.x % width;
  for (int g = blockIdx.x * per + threadIdx.x / width; g < G; g += (gridDim.x - STATS) * per) {
    const int gf = a.ginfo[3 * g], gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    const int2 b = a.gblocks[g];
    if (u >= gc || b.y < 0) continue;
    const double *q = a.psum + 4 * ((int64_t)b.x * a.n_crit + u);
    const int64_t step = 4 * (int64_t)a.n_crit;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k = 0; k < b.y; ++k, q += step) {
      const double2 x = reinterpret_cast<const double2 *>(q)[0], y = reinterpret_cast<const double2 *>(q)[1];
      v[0] += x.x;
      v[1] += x.y;
      v[2] += y.x;
      v[3] += y.y;
    }
    const int i = gf + u;
    const double eps = a.par[gs].eps;
    const double self = self_potential(a.smass[i], (float)(eps * eps));
    const int o = a.perm[i];
    a.acc[3 * (int64_t)o] = (float)v[0];
    a.acc[3 * (int64_t)o + 1] = (float)v[1];
    a.acc[3 * (int64_t)o + 2] = (float)v[2];
    a.pot[o] = (float)(self - v[3]);
  }
}

// Before the next outliers: their counters.  again: the same ones in a larger
// pool.
__global__ void k_next_outliers(DevInfo *info, bool again) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  info->queue = 0;
  info->queue2 = 0;
  info->blocks_done = max(info->blocks_done, info->blocks);
  info->blocks = 0;
  info->rows = 0;
  if (again) info->err &= ~kErrPool;
  else info->tasks_done += info->tasks;
  info->tasks = 0;
}

// Outliers: 4 members per workgroup, 64 threads per member, each adding the
// rows of a 64th of the tasks in order; the parts are added in order after the
// group's own rows.  The first workgroup of an outlier also adds up its list
// length and mass and the list statistics.  (Bound by the chain of a task: its record, then its rows; with
// 16 parts the outliers of a 64-system batch took 230 us, with 64 under 100.)
__global__ __launch_bounds__(256) void k_task_reduce(WideArgs a) {
  __shared__ double part[64][4][4];
  __shared__ double pm[256];
  __shared__ int4 pl[4];
  if (a.info->err & (kErrPool | kErrWide)) return;
  const int nout = min(a.info->n_out - a.out_first, a.lot);
  const int u = threadIdx.x & 3, sl = threadIdx.x >> 2;
  const int64_t step = 4 * (int64_t)a.n_crit;
  for (int o = blockIdx.y; o < nout; o += gridDim.y) {
    const OutInfo I = a.outinfo[o];
    const int gf = a.ginfo[3 * I.g], gc = a.ginfo[3 * I.g + 1], gs = a.ginfo[3 * I.g + 2];
    const int i = blockIdx.x * 4 + u;
    if ((int)blockIdx.x * 4 >= gc) continue;  // (the whole workgroup)
    const int t0 = (int)((int64_t)I.tasks * sl / 64), t1 = (int)((int64_t)I.tasks * (sl + 1) / 64);
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (sl == 0 && i < gc)
      for (int k = 0; k < I.rows; ++k) {
        const double *q = a.psum + (I.row0 + k) * step + 4 * i;
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] += q[c];
      }
#pragma unroll 2
    for (int k = t0; k < t1; ++k) {
      const int4 r = a.trows[I.task0 + k];
      if (i < gc)
        for (int j = 0; j < r.y; ++j) {
          const double *q = a.psum + (r.x + j) * step + 4 * i;
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] += q[c];
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) part[sl][u][c] = v[c];
    if (blockIdx.x == 0) {
      // list length, mass and statistics: each thread a run of the tasks, the
      // masses added in order
      const int k0 = (int)((int64_t)I.tasks * threadIdx.x / 256), k1 = (int)((int64_t)I.tasks * (threadIdx.x + 1) / 256);
      double mass = 0.0;
      int len = 0, visits = 0, near = 0;
      for (int k = k0; k < k1; ++k) {
        const int4 r = a.trows[I.task0 + k];
        len += r.z;
        visits += r.w;
        near += a.tnear[I.task0 + k];
        mass += a.tmass[I.task0 + k];
      }
      pm[threadIdx.x] = mass;
      const int lane = lane_id(), wv = threadIdx.x / kWave;
      len = wave_inclusive_sum(len);
      visits = wave_inclusive_sum(visits);
      near = wave_inclusive_sum(near);
      if (lane == kWave - 1) pl[wv] = make_int4(len, visits, near, 0);
    }
    __syncthreads();
    if (sl == 0 && i < gc) {
      for (int k = 1; k < 64; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] += part[k][u][c];
      const double eps = a.par[gs].eps;
      const double self = self_potential(a.smass[gf + i], (float)(eps * eps));
      const int64_t d = a.perm[gf + i];
      a.acc[3 * d] = (float)v[0];
      a.acc[3 * d + 1] = (float)v[1];
      a.acc[3 * d + 2] = (float)v[2];
      a.pot[d] = (float)(self - v[3]);
    }
    if (blockIdx.x == 0 && threadIdx.x < kWave) {
      double m = I.mass;
      for (int k = 0; k < 256; ++k) m += pm[k];
      int total = I.len, visits = I.visits, near = I.near;
      for (int w = 0; w < 4; ++w) {
        total += pl[w].x;
        visits += pl[w].y;
        near += pl[w].z;
      }
      if (threadIdx.x == 0) {
        a.glist[I.g] = total;
        a.gmass[I.g] = m;
      }
      ListStats st;
      if (threadIdx.x == 0) st.add(gc, total, visits, near);
      st.store(a.info);
    }
    __syncthreads();
  }
}

}  // namespace

int wide_block_length(int64_t n) {
  int bl = 256;
  while (bl < kMaxTile && (int64_t)bl * 1024 < n) bl *= 2;
  return bl;
}

bool wide_fits(int64_t n) { return 3 * ((n + wide_block_length(n) - 1) / wide_block_length(n)) + 2 <= kWideIds; }

// Threads per group, from the expected number of groups (a group holds about
// two thirds of n_crit): as many as keep every compute unit busy in one round.
static int wide_threads(int64_t n, int n_crit, int num_cu) {
  const int64_t groups = 3 * n / (2 * (int64_t)n_crit) + 1;
  return groups <= num_cu ? 1024 : (groups <= 2 * num_cu ? 512 : 256);
}

template <int NT, int MODE>
static void launch_walk_wide(const WideArgs &a, int grid, hipStream_t s) {
  if constexpr (MODE == kUnitGroups) {  // (only with quadrupoles)
    k_walk_wide<NT, true, MODE><<<(unsigned)grid, NT, 0, s>>>(a);
  } else {
    if (a.slot)
      k_walk_wide<NT, true, MODE><<<(unsigned)grid, NT, 0, s>>>(a);
    else
      k_walk_wide<NT, false, MODE><<<(unsigned)grid, NT, 0, s>>>(a);
  }
}

void walk_wide_device(const WideArgs &a, int64_t n, int num_cu, hipStream_t s) {
  switch (wide_threads(n, a.n_crit, num_cu)) {
    case 1024: launch_walk_wide<1024, kUnitGroups>(a, num_cu, s); break;
    case 512: launch_walk_wide<512, kUnitGroups>(a, 2 * num_cu, s); break;
    default: launch_walk_wide<256, kUnitGroups>(a, 5 * num_cu, s);
  }
}

void walk_outliers_device(const WideArgs &a, hipStream_t s) { launch_walk_wide<1024, kUnitOutliers>(a, a.lot, s); }

void next_outliers_device(DevInfo *info, bool again, hipStream_t s) { k_next_outliers<<<1, 64, 0, s>>>(info, again); }

void walk_tasks_device(const WideArgs &a, int num_cu, hipStream_t s) {
  launch_walk_wide<256, kUnitTasks>(a, kTaskGroups * num_cu, s);
}

void force_blocks_device(const WideArgs &a, int num_cu, hipStream_t s) {
  const unsigned grid = (unsigned)(num_cu * 6);
  if (a.slot)
    k_force_blocks<true><<<grid, 256, 0, s>>>(a);
  else
    k_force_blocks<false><<<grid, 256, 0, s>>>(a);
}

void block_reduce_device(const WideArgs &a, int num_cu, bool stats, hipStream_t s) {
  const int width = a.n_crit <= 64 ? 64 : (a.n_crit <= 128 ? 128 : 256);
  if (stats)
    k_block_reduce<true><<<(unsigned)(num_cu * 8 + 1), 256, 0, s>>>(a, width);
  else
    k_block_reduce<false><<<(unsigned)(num_cu * 8), 256, 0, s>>>(a, width);
}

void task_reduce_device(const WideArgs &a, hipStream_t s) {
  k_task_reduce<<<dim3((unsigned)((a.n_crit + 3) / 4), 32), 256, 0, s>>>(a);
}

}  // namespace bh
