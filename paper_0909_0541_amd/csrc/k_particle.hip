// Per-particle walk: the paper's own GPU form (Fig. "treegpu", Sec. 3.4), where
// each particle opens and accepts nodes by itself and sums what it accepts,
// with no shared list.
//
// The opening test is the group test with the group reduced to the particle (a
// point box): d^2 = |com - x_i|^2 (FP64) against (l/theta + s)^2 (Eq. 2/3), so
// the terms summed are those of the lists of one-particle groups.  A particle
// skips itself.  Terms are summed in FP32 from the FP64 relative vector (x_j -
// x_i rounded once), folded into FP64 every kDrain terms at most.
//
// One wave walks for a bundle of P neighbouring particles (in key order, of
// one system): a node that any of them reaches is read and tested once, with
// the mask of the particles that reach it.  The bundle's box settles most
// tests: rounding is monotone, so if the box's nearest point is beyond the
// opening distance every particle's own test accepts, and if its farthest
// point is within it every one opens.  The others are tested particle by
// particle, 64 / P nodes at a time.  Accepted nodes go to LDS with the mask of
// the particles that take them and are summed from there, 64 / P at a time.
//
// Bound by vector issue (81 % of the launch's cycles, sphere of 200,003; half for
// terms, about 20 instructions each, half for tests and bookkeeping).  With one lane per walk
// over a threaded tree, each visit waiting for its node's 64 bytes: sphere of
// 200,003 particles 1411 us, with this 343; clustered box of 2M 46.4 and 5.1
// ms.
#include "bh_device.h"

namespace bh {

namespace {

// Particles of a bundle.  More share a node's test but take fewer of the
// bundle's accepted nodes each; with few particles the shorter walks of more
// waves win (us with 16 and with 32: 3000 Plummer particles 85 and 130, 30,000
// 163 and 220, sphere of 200,003 343 and 381, clustered box of 300,000 787 and
// 780, of 2M 5490 and 5096).
constexpr int kFewBundle = 16, kBundle = 32;
constexpr int64_t kFewParticles = 1 << 18;
constexpr int kStack = 320;     // ranges of children to visit
constexpr int kReserve = 32;    // of these for a walk of one node at a time (a range a level)
constexpr int kDrain = 64;      // entries summed at a time

template <int P>
struct Lds {
  int2 range[kStack];           // first node, nodes
  uint32_t mask[kStack];        // particles that reach them
  double x[2 * kDrain], y[2 * kDrain], z[2 * kDrain];  // entries
  float m[2 * kDrain];
  uint32_t taken[2 * kDrain];   // particles that take them
  double q2[kWave];             // opening distances squared (nodes tested particle by particle)
  int32_t pick[kWave];
};

struct Acc {
  float ax = 0.f, ay = 0.f, az = 0.f, pt = 0.f;
  double dx = 0.0, dy = 0.0, dz = 0.0, dp = 0.0;
  int len = 0;
};

// Entries [e0, e1), every K-th from this lane's part on.
template <int P>
__device__ __forceinline__ void drain(Acc &A, const Lds<P> &L, int e0, int e1, int part, int u, double x0, double x1,
                                      double x2, float eps2) {
  constexpr int K = kWave / P, U = 4;
  auto one = [&](int e, bool on) {
    const int bit = on ? __builtin_amdgcn_sbfe((int)L.taken[e], u, 1) : 0;  // -1: takes it
    const float m = __int_as_float(__float_as_int(L.m[e]) & bit);
    const float dx = (float)__dsub_rn(L.x[e], x0), dy = (float)__dsub_rn(L.y[e], x1),
                dz = (float)__dsub_rn(L.z[e], x2);
    float q = __builtin_fmaf(dx, dx, eps2);
    q = __builtin_fmaf(dy, dy, q);
    q = __builtin_fmaf(dz, dz, q);
    const float ri = __builtin_amdgcn_rsqf(q);
    const float mr = m * ri;
    const float f = mr * (ri * ri);
    A.ax = __builtin_fmaf(f, dx, A.ax);
    A.ay = __builtin_fmaf(f, dy, A.ay);
    A.az = __builtin_fmaf(f, dz, A.az);
    A.pt += mr;
    A.len -= bit;
  };
  int e = e0;
  for (; e + U * K <= e1; e += U * K) {
#pragma unroll
    for (int k = 0; k < U; ++k) one(e + k * K + part, true);
  }
  for (; e < e1; e += K) one(min(e + part, e1 - 1), e + part < e1);
  A.dx += (double)A.ax;
  A.dy += (double)A.ay;
  A.dz += (double)A.az;
  A.dp += (double)A.pt;
  A.ax = A.ay = A.az = A.pt = 0.f;
}

template <int P>
__global__ __launch_bounds__(kWave) void k_pp_forces(const NodeRec *__restrict__ nodes, const SysInfo *__restrict__ sys,
                                                     int nsys, const SysParam *__restrict__ par,
                                                     const double *__restrict__ spos, const int32_t *__restrict__ perm,
                                                     int64_t n, float *__restrict__ acc, float *__restrict__ pot,
                                                     int4 *__restrict__ stat, DevInfo *__restrict__ info) {
  constexpr int K = kWave / P;
  __shared__ Lds<P> L;
  const int lane = lane_id(), u = lane % P, part = lane / P;
  // bundle b of system s is workgroup first / P + s + b: room for every
  // system's last, partly filled bundle
  int s = 0;
  {
    int lo = 0, hi = nsys - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (sys[mid].first / P + mid <= (int)blockIdx.x) lo = mid;
      else hi = mid - 1;
    }
    s = lo;
  }
  const int i0 = sys[s].first + ((int)blockIdx.x - (sys[s].first / P + s)) * P;
  const int cnt = min(P, sys[s].first + sys[s].count - i0);
  if (cnt <= 0) {
    if (lane == 0) stat[blockIdx.x] = make_int4(0, 0, 0, 0);
    return;
  }
  const int nslots = nsys + info->n_slots;
  const int i = i0 + min(u, cnt - 1);  // (a lane without a particle: the last one's position, in no mask)
  const double x0 = spos[3 * (int64_t)i], x1 = spos[3 * (int64_t)i + 1], x2 = spos[3 * (int64_t)i + 2];
  double lo[3] = {x0, x1, x2}, hi[3] = {x0, x1, x2};
#pragma unroll
  for (int d = 1; d < P; d <<= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = fmin(lo[k], shfl_xor_d(lo[k], d));
      hi[k] = fmax(hi[k], shfl_xor_d(hi[k], d));
    }
  const double eps = par[s].eps, theta = par[s].theta;
  const float eps2 = (float)(eps * eps);
  // l / theta = (side / theta) * 2^-level exactly, as in the group walk
  const double side = sys[s].side, side_theta = side / theta;
  const int side_exp = ilogb(side);
  Acc A;
  uint32_t own = 0;  // particles whose own leaf was reached
  if (lane == 0) {
    L.range[0] = make_int2(s, 1);
    L.mask[0] = (uint32_t)((2ull << (cnt - 1)) - 1ull);
  }
  int sp = 1, nb = 0;
  int guard = 2 * nslots + 4;
  __syncthreads();
  while (sp > 0) {
    if (--guard < 0) {
      if (lane == 0) atomicOr(&info->err, kErrStack);
      break;
    }
    // the next nodes: of the topmost ranges, 64 at most, fewer when the ranges
    // of their children might not fit
    const int limit = max(1, min(kWave, kStack - kReserve - sp));
    const int at = sp - 1 - lane;
    const int2 rg = L.range[max(at, 0)];
    const int rc = at >= 0 ? min(rg.y, kWave) : 0;
    const int inc = wave_inclusive_sum(rc), off = inc - rc;
    const int total = min(limit, __builtin_amdgcn_readlane(inc, kWave - 1));
    L.pick[lane] = 0;
    __syncthreads();
    if (rc > 0 && off < limit) L.pick[off] = lane;
    __syncthreads();
    const int r = wave_inclusive_max(L.pick[lane]);
    const bool on = lane < total;
    const int roff = __shfl(off, r, kWave), rat = max(sp - 1 - r, 0);
    const int v = L.range[rat].x + (lane - roff);
    const uint32_t mk = on ? L.mask[rat] : 0u;
    const int gone = __popcll(__ballot(at >= 0 && off + rg.y <= limit));
    __syncthreads();
    if (at >= 0 && off < limit && off + rg.y > limit) L.range[at] = make_int2(rg.x + (limit - off), rg.y - (limit - off));
    sp -= gone;
    // tests
    uint32_t take = 0, open = 0, rest = 0;
    NodeRec nd;
    nd.child = -1;
    nd.nchild = 0;
    nd.m = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) nd.com[k] = 0.0;
    double q2 = 0.0;
    if (on && v >= 0 && v < nslots) {
      nd = nodes[v];
      if (nd.child < 0) {
        const int d = nd.first - i0;
        const uint32_t self = (d >= 0 && d < P) ? 1u << d : 0u;
        own |= mk & self;
        take = mk & ~self;
      } else {
        double q = isfinite(nd.l) ? ldexp(side_theta, ilogb(nd.l) - side_exp) : nd.l;
        q = __dadd_rn(q, nd.s);
        q2 = __dmul_rn(q, q);
        double dn = 0.0, df = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double a = __dsub_rn(lo[k], nd.com[k]), b = __dsub_rn(nd.com[k], hi[k]);
          const double en = fmax(0.0, fmax(a, b)), ef = fmax(-a, -b);
          dn = (k == 0) ? __dmul_rn(en, en) : __dadd_rn(dn, __dmul_rn(en, en));
          df = (k == 0) ? __dmul_rn(ef, ef) : __dadd_rn(df, __dmul_rn(ef, ef));
        }
        if (dn > q2) take = mk;
        else if (df <= q2) open = mk;
        else rest = mk;
      }
    } else if (on) {
      atomicOr(&info->err, kErrStack);
    }
    unsigned long long todo = __ballot(rest != 0);
    if (todo) {
      if (rest) {  // (places beyond the entries waiting: fewer than kDrain)
        L.x[kDrain + lane] = nd.com[0];
        L.y[kDrain + lane] = nd.com[1];
        L.z[kDrain + lane] = nd.com[2];
        L.q2[lane] = q2;
      }
      __syncthreads();
      while (todo) {
        int node[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          node[k] = todo ? __ffsll(todo) - 1 : -1;
          todo &= todo - 1;
        }
        int mine = node[0];
#pragma unroll
        for (int k = 1; k < K; ++k) mine = part == k ? node[k] : mine;
        const int w = max(mine, 0);
        const double e0 = __dsub_rn(L.x[kDrain + w], x0), e1 = __dsub_rn(L.y[kDrain + w], x1),
                     e2 = __dsub_rn(L.z[kDrain + w], x2);
        const double d2 = __dadd_rn(__dadd_rn(__dmul_rn(e0, e0), __dmul_rn(e1, e1)), __dmul_rn(e2, e2));
        const unsigned long long far = __ballot(d2 > L.q2[w]);
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (lane == node[k]) {
            const uint32_t f = (uint32_t)(far >> (k * P)) & (uint32_t)((2ull << (P - 1)) - 1ull);
            take = rest & f;
            open = rest & ~f;
          }
      }
      __syncthreads();
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned long long tb = __ballot(take != 0), ob = __ballot(open != 0 && nd.nchild > 0);
    if (take) {
      const int e = nb + __popcll(tb & below);
      L.x[e] = nd.com[0];
      L.y[e] = nd.com[1];
      L.z[e] = nd.com[2];
      L.m[e] = (float)nd.m;
      L.taken[e] = take;
    }
    if (open != 0 && nd.nchild > 0) {
      const int t = sp + __popcll(ob & below);
      L.range[t] = make_int2(nd.child, nd.nchild);
      L.mask[t] = open;
    }
    nb += __popcll(tb);
    sp += __popcll(ob);
    __syncthreads();
    if (nb >= kDrain) {
      drain<P>(A, L, nb - kDrain, nb, part, u, x0, x1, x2, eps2);
      nb -= kDrain;
      __syncthreads();
    }
  }
  drain<P>(A, L, 0, nb, part, u, x0, x1, x2, eps2);
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) own |= __shfl_xor((int)own, d, kWave);
#pragma unroll
  for (int d = P; d < kWave; d <<= 1) {
    A.dx += shfl_xor_d(A.dx, d);
    A.dy += shfl_xor_d(A.dy, d);
    A.dz += shfl_xor_d(A.dz, d);
    A.dp += shfl_xor_d(A.dp, d);
    A.len += __shfl_xor(A.len, d, kWave);
  }
  // a particle's list, as the one-particle group would hold it: the entries
  // taken plus its own leaf when the walk reached it (not an interaction)
  int len = 0;
  if (part == 0 && u < cnt) {
    len = A.len + (int)((own >> u) & 1u);
    const int64_t o = perm[i];
    acc[3 * o] = (float)A.dx;
    acc[3 * o + 1] = (float)A.dy;
    acc[3 * o + 2] = (float)A.dz;
    pot[o] = (float)(-A.dp);
  }
  int inter = max(len - 1, 0), entries = len, longest = len;
#pragma unroll
  for (int d = 1; d < P; d <<= 1) {
    inter += __shfl_xor(inter, d, kWave);
    entries += __shfl_xor(entries, d, kWave);
    longest = max(longest, __shfl_xor(longest, d, kWave));
  }
  if (lane == 0) stat[blockIdx.x] = make_int4(inter, entries, longest, 0);
}

// List statistics of all bundles (an atomic per bundle and counter, all on one
// line, would take longer than the walk).
__global__ __launch_bounds__(1024) void k_pp_stats(const int4 *__restrict__ stat, int count, DevInfo *info) {
  unsigned long long inter = 0, entries = 0;
  int longest = 0;
#pragma unroll 4
  for (int k = threadIdx.x; k < count; k += 1024) {
    const int4 v = stat[k];
    inter += (uint32_t)v.x;
    entries += (uint32_t)v.y;
    longest = max(longest, v.z);
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    inter += __shfl_xor(inter, d, kWave);
    entries += __shfl_xor(entries, d, kWave);
    longest = max(longest, __shfl_xor(longest, d, kWave));
  }
  if (lane_id() == 0 && entries) {
    atomicAdd(&info->interactions, inter);
    atomicAdd(&info->list_entries, entries);
    atomicMax(&info->max_list, longest);
  }
}

}  // namespace

static int bundle(int64_t n) { return n <= kFewParticles ? kFewBundle : kBundle; }

size_t particle_stat_bytes(int64_t n, int nsys) { return sizeof(int4) * (size_t)(n / bundle(n) + nsys + 1); }

void particle_forces_device(const NodeRec *nodes, int nsys, const SysInfo *sys, const SysParam *par,
                            const double *spos, const int32_t *perm, int64_t n, float *acc, float *pot, int4 *stat,
                            DevInfo *info, hipStream_t s) {
  if (n <= 0) return;
  const int P = bundle(n), blocks = (int)(n / P) + nsys + 1;
  if (P == kFewBundle)
    k_pp_forces<kFewBundle><<<(unsigned)blocks, kWave, 0, s>>>(nodes, sys, nsys, par, spos, perm, n, acc, pot, stat,
                                                               info);
  else
    k_pp_forces<kBundle><<<(unsigned)blocks, kWave, 0, s>>>(nodes, sys, nsys, par, spos, perm, n, acc, pot, stat, info);
  k_pp_stats<<<1, 1024, 0, s>>>(stat, blocks, info);
}

}  // namespace bh
