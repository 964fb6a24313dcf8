// Neighbour search and SPH density: the general treewalk of Sec. 3.3 (Fig.
// "general_treewalk") applied to a short-range interaction, as in smoothed
// particle hydrodynamics, the application the paper names.
//
// The neighbours of particle i are the particles j != i with |x_j - x_i| <
// h_i, its own search radius (the "gather" form).  The walk is the group form
// used for gravity: one wavefront per group, persistent grid pulling groups
// from an atomic queue, up to 64 nodes tested per iteration from a stack of
// slot ranges in LDS.  The distance test of the general walk prunes a cell
// whose particles all lie farther than the group's largest radius from the
// group's bounding box: every particle of a cell lies within
// (sqrt(3)/2) l + s of its centre of mass (l the cube side, s the distance of
// the centre of mass from the cube's centre).  A particle leaf within that
// radius of the box is a candidate; candidates collect in LDS and are
// tested against every member: an FP32 scan marks the possible neighbours, and
// what is marked is decided in FP64 with the squared distance (dx^2 + dy^2) +
// dz^2 rounded as written, so the decision r^2 < h_i^2 is the same as a plain
// CPU evaluation.  The pruning bounds carry margins far above FP64 rounding;
// they only skip work, the per-pair test decides.
//
// Outliers.  A group in a sparse place has a large search radius and may have
// nearly every particle for a candidate, hundreds of times the median, while
// the other waves are done.  A walk that finds cells inside its radius which
// together hold out_min particles gives its group up at once to a second
// launch, in which up to kNbSlices waves search a part of the particles each
// (consecutive in key order; nodes without any are pruned); their counts and
// sums are added in order.  30,000 Plummer particles: 6.4 ms with a wave for
// each group, 0.99 ms like this; 300,000 in groups of 128 46 and 4.2 ms.  (Not
// for calls that ask for lists, whose order is the walk's.)
//
// The SPH density sums m_j W(r_ij, h_i) over the neighbours, plus the
// particle's own m_i W(0, h_i), with the cubic spline kernel of Monaghan and
// Lattanzio with compact support h (the paper fixes no kernel).  Lists, when
// asked for, hold the input indices of the neighbours in walk order.
#include <algorithm>
#include <type_traits>

#include "bh_device.h"

namespace bh {

namespace {

constexpr int kNbStack = 512;                    // range stack entries
constexpr int kNbReserve = 8 * 24;               // growth bound in one-range mode
// Particles of a cell that is not opened (1M clustered particles in groups of 8,
// 32 and 64, radii of the mean distance, us: 64 2472, 1019, 732; 128 2468, 983,
// 712; 256 2706, 1052, 746; 512 3031, 1143, 790).
constexpr int kNbRun = 128;
// Particles of cells inside the radius that make an outlier: a sixteenth of
// all, at least kNbOutMin.  (8192 for 1M clustered particles makes outliers of
// a few hundred groups that end in time: 3.14 ms against 2.61.)
constexpr int kNbOutMin = 4096;
constexpr int kNbSlices = 64;                    // parts of an outlier's search,
constexpr int kNbSliceMin = 1024;                // of at least so many particles
constexpr int kNbRows = 256 * kNbSlices;         // parts of all outliers
constexpr int kNbCand = 128;                     // candidate buffer: 64 to test and 64 that a batch may add
// Marks per candidate beyond which the members test the candidates one after
// another instead (flush): with densities, counts only, and with lists, whose
// rows the members then write at 64 places rather than run by run.  30,000
// clustered particles with 1855 neighbours each in groups of 64, us: 1718 and 703,
// always in rounds 5016 and 3237; a sphere of 1M, 209 neighbours: 1834 and 1217,
// with 10 and 4 here 1911 and 1239, with 20 and 12 1847 and 1252.  Lists of 128,052
// Plummer particles in groups of 128 (42 neighbours) and of 139,809 in groups of 32
// (71), ms: always in rounds 23.2 and 35.5, from 14 on 26.3 and 29.1, 20 23.0 and
// 29.3, 28 23.1 and 33.9.
constexpr int kDenseSum = 14, kDenseCount = 8, kDenseList = 20;
constexpr double kHalfSqrt3 = 0.86602540378443865;

__device__ __forceinline__ void wave_sync() { __syncthreads(); }

// The kernel at q = r / h < 1, over sigma = 8 / (pi h^3); both branches
// without a jump.
__device__ __forceinline__ double sph_sigma(double h) { return 8.0 / (3.14159265358979323846 * h * h * h); }
__device__ __forceinline__ double sph_shape(double q) {
  const double u = 1.0 - q;
  const double in = 1.0 - 6.0 * q * q + 6.0 * q * q * q;
  const double out = 2.0 * u * u * u;
  return q < 0.5 ? in : (q < 1.0 ? out : 0.0);
}

// sqrt(r2) / h from the hardware estimate of 1 / sqrt(r2) and hi = 1 / h, each
// with one residual step, so that square root and quotient are rounded as the
// library's to within a few hundredths of an ulp.  For h in (2^-400, 2^400)
// and r2 < h^2; below 2^-900, r2 counts as that (the kernel is flat to 1e-30
// there).
__device__ __forceinline__ double ratio(double r2, double h, double hi) {
  r2 = fmax(r2, 0x1p-900);
  const double y0 = __builtin_amdgcn_rsq(r2);
  const double e = __builtin_fma(-(r2 * y0), y0, 1.0);
  const double y = __builtin_fma(y0 * e, __builtin_fma(0.375, e, 0.5), y0);
  double r = r2 * y;
  r = __builtin_fma(0.5 * y, __builtin_fma(-r, r, r2), r);
  double q = r * hi;
  return __builtin_fma(__builtin_fma(-q, h, r), hi, q);
}

__global__ void k_nb_reset(DevInfo *info) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    info->queue = 0;
    info->nb_pairs = 0;
    info->nb_tests = 0;
    info->nb_out = 0;
    info->nb_queue = 0;
  }
}

// Candidates staged in LDS: position and mass (taken from the particle's node
// record by the lane that accepted it), and for the scan the position
// relative to the group's centre in FP32, with the sorted index.
struct alignas(16) CandRec {
  double x, y, z, m;
};
struct Cand {
  CandRec c[kNbCand];
  float4 f[kNbCand];  // scan frame: -2 x, -2 y, -2 z, |x|^2
  int32_t j[kNbCand]; // sorted index
  unsigned long long words[kWave];  // marks of the scan
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t __attribute__((may_alias)) Piece;  // a quarter of a mark word

// 2 v plus this lane's bit of mask, in one instruction.
__device__ __forceinline__ uint32_t shift_in(uint32_t v, unsigned long long mask) {
  uint32_t r;
  asm("v_addc_co_u32_e64 %0, vcc, %1, %1, %2" : "=v"(r) : "v"(v), "s"(mask) : "vcc");
  return r;
}

// Position of the r-th set bit (r counted from 0) of a word with more than r.
__device__ __forceinline__ int nth_bit(unsigned long long w, int r) {
  uint32_t x = (uint32_t)w;
  int at = 0;
  const int lo = __popc(x);
  if (r >= lo) {
    r -= lo;
    x = (uint32_t)(w >> 32);
    at = 32;
  }
#pragma unroll
  for (int half = 16; half > 0; half >>= 1) {
    const int n = __popc(x & ((1u << half) - 1u));
    const bool up = r >= n;
    r -= up ? n : 0;
    at += up ? half : 0;
    x = up ? x >> half : x;
  }
  return at;
}

// Inclusive sums over runs of lanes: lane l adds the values of lanes
// first .. l (first <= l, the same on all lanes of a run).  The steps are
// those of wave_inclusive_sum, each taken where the lanes it brings in belong
// to the run.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const int2 a = *reinterpret_cast<int2 *>(&v);
  int2 b;
  b.x = __builtin_amdgcn_mov_dpp(a.x, CTRL, 0xf, 0xf, true);
  b.y = __builtin_amdgcn_mov_dpp(a.y, CTRL, 0xf, 0xf, true);
  return *reinterpret_cast<double *>(&b);
}
template <int CTRL>
__device__ __forceinline__ double run_step(double v, bool on) {
  const double u = dpp_d<CTRL>(v);
  return __dadd_rn(v, on ? u : 0.0);
}
__device__ __forceinline__ double run_sum(double v, int first, int lane) {
  const int back = lane - first, in_row = min(back, lane & 15);  // lanes of the run below this one
  v = run_step<kDppRowShr1>(v, in_row >= 1);
  v = run_step<kDppRowShr2>(v, in_row >= 2);
  v = run_step<kDppRowShr4>(v, in_row >= 4);
  v = run_step<kDppRowShr8>(v, in_row >= 8);
  v = run_step<kDppRowBcast15>(v, (lane & 16) && back > (lane & 15));
  return run_step<kDppRowBcast31>(v, lane >= 32 && first < 32);
}

// The candidates one after another, a member per lane (h2 = 0 and no index on a
// lane without one), U at a time.  Where most pairs are neighbours: 13
// instructions a candidate for the count and 40 with the density, whatever the
// number of hits, against some 110 and 180 a round of 64 marked pairs.
template <int U, bool RHO, bool LISTS>
__device__ __forceinline__ void direct(const NeighborArgs &a, const Cand &cd, int nc, int i, double x0, double x1,
                                       double x2, double h, double h2, double hi, double sigma, bool plain, int64_t row,
                                       int64_t len, int &c, double &r) {
  auto terms = [&](auto n, int k0) {
    constexpr int N = decltype(n)::value;
    CandRec q[N];
    int j[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      q[u] = cd.c[k0 + u];
      j[u] = cd.j[k0 + u];
    }
    double r2[N];
    bool hit[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const double dx = __dsub_rn(q[u].x, x0), dy = __dsub_rn(q[u].y, x1), dz = __dsub_rn(q[u].z, x2);
      r2[u] = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
      hit[u] = r2[u] < h2 && j[u] != i;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if (LISTS && hit[u] && c < len) a.nbr[row + c] = a.perm[j[u]];
      c += hit[u] ? 1 : 0;
    }
    if (RHO) {
      double W[N];
#pragma unroll
      for (int u = 0; u < N; ++u)
        W[u] = __dmul_rn(q[u].m, sigma * sph_shape(plain ? ratio(r2[u], h, hi) : sqrt(r2[u]) / h));
#pragma unroll
      for (int u = 0; u < N; ++u) r = __dadd_rn(r, hit[u] ? W[u] : 0.0);
    }
  };
  int k = 0;
  for (; k + U <= nc; k += U) terms(std::integral_constant<int, U>{}, k);
  for (; k < nc; ++k) terms(std::integral_constant<int, 1>{}, k);
}

// Tests the first nc <= 64 staged candidates against every member block.
//
// About one pair in fifteen is a neighbour pair, in nearly every candidate
// some lane has one, and the lane with the most has several times the mean.
// Testing and adding candidate by candidate (or each lane its own hits) made
// the wave run the FP64 kernel function for nearly every candidate.  So:
//   scan   marks the possible neighbours by |x|^2 - 2 x.y against a bound
//          less |y|^2 (x candidate, y member, FP32 in the group's frame) that
//          no rounding can exceed (a superset; NaN marks): 16 candidates times
//          16 members, four terms, is one matrix instruction, so the vector
//          units only compare and shift the marks in.
//   rounds the marked (member, candidate) pairs, counted member by member, are
//          taken 64 at a time, one per lane whoever's member it is: the FP64
//          decision (r2 < h2, the sum rounded as written), the density term,
//          and the sum over each member's run of lanes.  Many marks: the
//          candidates one after another (direct).
// 1,048,576 clustered particles, 133 neighbours and 1874 tests a particle:
// 5.9 ms testing and adding candidate by candidate, 5.3 ms with the pairs
// listed in LDS and each member adding its terms one after another, 2.99 ms
// in rounds, 2.84 ms without visiting the leaves (then bound by vector issue at
// 87 %), 2.52 ms with the scan on the matrix units (before, nine vector
// instructions a candidate and wave).  Now vector issue takes 69 % of the
// cycles of a compute unit that has waves (three a SIMD), most of it the rounds,
// about 180 instructions each.
template <int kNbBlocks, bool RHO, bool LISTS>
__device__ __forceinline__ void flush(const NeighborArgs &a, Cand &cd, int *mark, int nc, int gf, int gc, int nb, int lane,
                                      const float (&fb)[kNbBlocks][4], const float (&ft)[kNbBlocks][4],
                                      const double (&hb)[kNbBlocks], int (&cb)[kNbBlocks], double (&rb)[kNbBlocks],
                                      const int64_t (&ob)[kNbBlocks], const int64_t (&lb)[kNbBlocks],
                                      bool plain, int &tests) {
#pragma unroll
  for (int b = 0; b < kNbBlocks; ++b) {
    if (b < nb) {
      const int i = gf + b * kWave + lane;
      const int m = min(gc - b * kWave, kWave);  // members of this block
      const bool live = lane < m;
      // scan: matrix row 4 q + i of tile t is candidate 16 q + 4 t + i, so
      // that lane 16 q + c ends with candidates 16 q ... 16 q + 15 of member c
      // of each member tile in order
      const float *fr = reinterpret_cast<const float *>(cd.f) + 4 * (16 * ((lane >> 2) & 3) + (lane & 3)) + (lane >> 4);
      const float row[4] = {fr[0], fr[16], fr[32], fr[48]};
      Piece *words = reinterpret_cast<Piece *>(cd.words);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (16 * w >= m) break;
        uint32_t got = 0;
#pragma unroll
        for (int t = 3; t >= 0; --t) {
          const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(row[t], fb[b][w], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
          for (int k = 3; k >= 0; --k) got = shift_in(got, __ballot(!(d[k] > ft[b][w])));
        }
        words[4 * (16 * w + (lane & 15)) + (lane >> 4)] = (Piece)got;
      }
      wave_sync();
      unsigned long long marks = cd.words[lane];
      // (places from nc on hold older candidates: their marks are cut off)
      if (nc < 64) marks &= (1ull << nc) - 1ull;
      if (!live) marks = 0ull;
      const int mine = __popcll(marks);
      const int off = wave_inclusive_sum(mine) - mine;
      const int total = __builtin_amdgcn_readlane(off + mine, kWave - 1);
      double x0 = 0.0, x1 = 0.0, x2 = 0.0;
      if (live) {
        x0 = a.spos[3 * (int64_t)i];
        x1 = a.spos[3 * (int64_t)i + 1];
        x2 = a.spos[3 * (int64_t)i + 2];
        tests += nc;
      }
      const double h = hb[b], hi = 1.0 / h;
      const double sigma = RHO ? sph_sigma(h) : 0.0;
      int c = cb[b];
      double r = rb[b];
      if (total > (LISTS ? kDenseList : RHO ? kDenseSum : kDenseCount) * nc) {
        constexpr int kU = RHO || kNbBlocks > 2 ? 2 : 4;  // (registers)
        direct<kU, RHO, LISTS>(a, cd, nc, live ? i : -1, x0, x1, x2, h, live ? __dmul_rn(h, h) : 0.0, hi, sigma, plain,
                               ob[b], lb[b], c, r);
        cb[b] = c;
        rb[b] = r;
        continue;
      }
      for (int q0 = 0; q0 < total; q0 += kWave) {
        // this lane's own pairs of the round are on lanes [s, e)
        const int s = min(max(off - q0, 0), kWave), e = min(max(off + mine - q0, 0), kWave);
        // lane's pair: the member whose run it lies in, and the candidate
        mark[lane] = 0;
        wave_sync();
        if (e > s) mark[s] = lane;
        wave_sync();
        const int u = wave_inclusive_max(mark[lane]);
        const bool have = q0 + lane < total;
        const int uoff = __shfl(off, u, kWave) - q0;
        const unsigned long long um = (unsigned long long)shfl_i64((int64_t)marks, u);
        const int k = have ? nth_bit(um, lane - uoff) : 0;
        const CandRec q = cd.c[k];
        const int j = cd.j[k];
        const double dx = __dsub_rn(q.x, shfl_d(x0, u));
        const double dy = __dsub_rn(q.y, shfl_d(x1, u));
        const double dz = __dsub_rn(q.z, shfl_d(x2, u));
        const double r2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
        const double hu = shfl_d(h, u);
        const bool hit = have && j != gf + b * kWave + u && r2 < __dmul_rn(hu, hu);
        const unsigned long long hits = __ballot(hit);
        if (LISTS) {
          // place in the member's row: the hits of its earlier pairs
          const unsigned long long before = ((1ull << lane) - 1ull) & ~((1ull << max(uoff, 0)) - 1ull);
          const int n0 = __shfl(c, u, kWave) + (int)__popcll(hits & before);
          const int64_t row = shfl_i64(ob[b], u), len = shfl_i64(lb[b], u);
          if (hit && n0 < len) a.nbr[row + n0] = a.perm[j];
        }
        if (RHO) {
          double x = 0.0;
          if (plain) x = ratio(r2, hu, shfl_d(hi, u));
          else x = sqrt(r2) / hu;
          const double W = shfl_d(sigma, u) * sph_shape(x);
          const double sum = shfl_d(run_sum(hit ? __dmul_rn(q.m, W) : 0.0, max(uoff, 0), lane), max(e - 1, 0));
          if (e > s) r = __dadd_rn(r, sum);
        }
        if (e > s) {
          const unsigned long long own = (e == kWave ? ~0ull : (1ull << e) - 1ull) & ~((1ull << s) - 1ull);
          c += (int)__popcll(hits & own);
        }
      }
      cb[b] = c;
      rb[b] = r;
    }
  }
}

// kNbBlocks: member blocks of 64 held per lane (the largest group / 64),
// chosen by the host from the grouping so that small groups keep registers
// free.  RUNS: a cell of at most kNbRun particles that is not pruned is not
// opened; its particles, consecutive in key order and with those of its
// neighbours in the batch one run, are read from the particle arrays, 64 at a
// time, and tested against the radius as their leaves would be, so the
// candidates are the same in another order.  Without (calls that ask for
// lists, whose order is the walk's) every leaf's 64-byte record is visited.
//
// SLICES: the launch for outliers, over the parts of info->nb_out groups.  RHO:
// densities too.  (With densities and lists chosen at run time a wave holds 10 to
// 60 registers more, and calls without dense blocks take 2 to 8 % longer.)
__device__ __forceinline__ int slices_per_outlier(int nout) {
  return nout <= kNbRows / kNbSlices ? kNbSlices : max(1, kNbRows / nout);
}
__device__ __forceinline__ int slices_of(int per, int count) { return max(1, min(per, count / kNbSliceMin)); }

template <int kNbBlocks, bool RUNS, bool SLICES, bool RHO>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(kNbBlocks == 1 ? 3 : 2))) void k_neighbors(NeighborArgs a) {
  __shared__ int2 stk[kNbStack];
  __shared__ Cand cd;
  __shared__ int mark[kWave];
  const int lane = lane_id();
  const int G = a.info->n_groups;
  const int nslots = a.nsys + a.info->n_slots;
  unsigned long long pairs = 0, all_tests = 0;
  const int per = SLICES ? slices_per_outlier(a.info->nb_out) : 1, units = SLICES ? a.info->nb_out * per : G;
  // (the first unit is the workgroup's own number: 3000 waves asking for one
  // on the same line take their time; 3000 particles 122 us against 86)
  for (int unit = blockIdx.x; unit < units;
       unit = (int)gridDim.x + take_one(SLICES ? &a.info->nb_queue : &a.info->queue, lane)) {
    const int g = SLICES ? a.out[unit / per] : unit;
    int tests = 0;
    const int gf = a.ginfo[3 * g], gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    const int nb = min((gc + kWave - 1) / kWave, kNbBlocks);
    if ((gc + kWave - 1) / kWave > kNbBlocks || gs < 0 || gs >= a.nsys) {
      if (lane == 0) atomicOr(&a.info->err, kErrStack);
      continue;
    }
    // this part's particles
    int p0 = 0, p1 = 0, parts = 1;
    if (SLICES) {
      const int sf = a.sys[gs].first, sn = a.sys[gs].count, k = unit % per;
      parts = slices_of(per, sn);
      if (k >= parts) continue;
      p0 = sf + (int)((int64_t)sn * k / parts);
      p1 = sf + (int)((int64_t)sn * (k + 1) / parts);
    }
    int inside = 0;  // particles in cells found inside the radius
    bool outlier = false;
    // members: radii, the group's largest, output offsets
    double hb[kNbBlocks], rb[kNbBlocks];
    int cb[kNbBlocks];
    int64_t ob[kNbBlocks], lb[kNbBlocks];
    double hmax = 0.0;
    bool bad = false, odd = false;
#pragma unroll
    for (int b = 0; b < kNbBlocks; ++b) {
      const int i = gf + b * kWave + lane;
      const bool live = b < nb && i < gf + gc;
      const int o = live ? a.perm[i] : 0;
      hb[b] = live ? a.h[o] : 1.0;
      if (live && !(hb[b] > 0.0 && hb[b] < INFINITY)) bad = true;
      if (!(hb[b] > 0x1p-400 && hb[b] < 0x1p400)) odd = true;
      if (live) hmax = fmax(hmax, hb[b]);
      cb[b] = 0;
      rb[b] = 0.0;
      ob[b] = 0;
      lb[b] = 0;
      if (!RUNS && live) {
        ob[b] = a.offsets[o];
        lb[b] = a.offsets[o + 1] - ob[b];
      }
    }
    if (__ballot(bad)) {
      if (lane == 0) atomicOr(&a.info->err, kErrRadius);
      continue;
    }
    const bool plain = __ballot(odd) == 0;  // radii of ordinary size
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) hmax = fmax(hmax, shfl_xor_d(hmax, d));
    // the group's box, widened by a margin above the rounding of the
    // distance sums, and the largest radius with a relative margin: a
    // neighbour of any member lies within rad of the box (a rounded box,
    // not the box grown into a cube)
    double elo[3], ehi[3], cpad = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double lo = a.gbox[6 * (int64_t)g + k], hi = a.gbox[6 * (int64_t)g + 3 + k];
      const double pad = 1e-15 * fmax(fabs(lo), fabs(hi)) + 1e-300;
      elo[k] = lo - pad;
      ehi[k] = hi + pad;
      cpad += pad;
    }
    const double rad = hmax * (1.0 + 1e-9) + cpad;
    // The scan's frame: positions relative to the box centre over a power of
    // two, so that coordinates of candidates and members are at most 2, and
    // FP32.  Of |x - y|^2 <= h^2 moved about as the scan has it, magnitudes
    // are at most 36; the roundings of coordinates, squares, four products and
    // their sum and the bound stay below 1.5e-5 (2^-15 is added).  A frame
    // beyond the ordinary range marks everything.
    double cen[3], ext = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cen[k] = 0.5 * (elo[k] + ehi[k]);
      ext = fmax(ext, 0.5 * (ehi[k] - elo[k]) + rad);
    }
    const bool ordinary = ext > 0x1p-900 && ext < 0x1p900;
    const double sc = ordinary ? ldexp(1.0, -ilogb(ext)) : 0.0;
    float fb[kNbBlocks][4], ft[kNbBlocks][4];
#pragma unroll
    for (int b = 0; b < kNbBlocks; ++b) {
      const int i = gf + b * kWave + lane;
      const bool live = b < nb && i < gf + gc;
      double y[3], yy = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        y[k] = live ? (a.spos[3 * (int64_t)i + k] - cen[k]) * sc : 0.0;
        yy += y[k] * y[k];
      }
      const double hs = hb[b] * sc;
      const float f0 = (float)y[0], f1 = (float)y[1], f2 = (float)y[2];
      const float lim = ordinary ? (float)(hs * hs * (1.0 + 1e-9) + 0x1p-15 - yy) : INFINITY;
      // member tile w's column: this lane holds component lane / 16 of member
      // 16 w + lane % 16
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int u = 16 * w + (lane & 15);
        const float c0 = __shfl(f0, u, kWave), c1 = __shfl(f1, u, kWave), c2 = __shfl(f2, u, kWave);
        fb[b][w] = lane < 16 ? c0 : (lane < 32 ? c1 : (lane < 48 ? c2 : 1.0f));
        ft[b][w] = __shfl(lim, u, kWave);
      }
    }

    int sp = 1, ncand = 0;
    if (lane == 0) stk[0] = make_int2(gs, 1);
    wave_sync();
    int budget = 4 * nslots + 4;
    // RUNS: a lane's particles [tf, te), the lanes that start a run, the lanes
    // that carry one on, and the run being read
    int tf = 0, te = 0, rp = 0, re = 0;
    unsigned long long heads = 0, inner = 0;
    while (sp > 0 || (RUNS && (heads || rp < re))) {
      if (--budget < 0) {
        if (lane == 0) atomicOr(&a.info->err, kErrStack);
        break;
      }
      bool push = false, is_cand = false;
      int2 rng = make_int2(0, 0);
      int j = 0;
      double px = 0.0, py = 0.0, pz = 0.0, pm = 0.0;
      if (RUNS && (heads || rp < re)) {
        if (rp >= re) {
          const int l0 = __ffsll((long long)heads) - 1;
          heads &= heads - 1;
          const unsigned long long rest = ~(inner >> l0 >> 1);
          rp = __builtin_amdgcn_readlane(tf, l0);
          re = __builtin_amdgcn_readlane(te, min(l0 + __ffsll((long long)rest) - 1, kWave - 1));
          if (rp < 0 || re > a.n) {
            if (lane == 0) atomicOr(&a.info->err, kErrStack);
            break;
          }
        }
        j = rp + lane;
        if (j < re) {
          px = a.spos[3 * (int64_t)j];
          py = a.spos[3 * (int64_t)j + 1];
          pz = a.spos[3 * (int64_t)j + 2];
          pm = a.smass[j];
          const double x[3] = {px, py, pz};
          double d2 = 0.0;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const double ek = fmax(0.0, fmax(elo[k] - x[k], x[k] - ehi[k]));
            d2 += ek * ek;
          }
          is_cand = d2 <= rad * rad;
        }
        rp += kWave;
      } else {
      // take up to 64 nodes from the top ranges (one range while the stack
      // is high: then the walk is depth first and the stack stays bounded)
      const bool starved = sp > kNbStack - kWave - kNbReserve;
      const int nread = starved ? 1 : min(sp, kWave);
      int2 e = make_int2(0, 0);
      if (lane < nread) e = stk[sp - 1 - lane];
      const int cnt = (lane < nread) ? e.y : 0;
      const int pre = wave_inclusive_sum(cnt);
      const int total = __shfl(pre, nread - 1, kWave);
      const int take = min(starved ? 8 : kWave, total);
      const int start = pre - cnt;
      const int kfull = __popcll(__ballot(lane < nread && pre <= take));
      mark[lane] = -1;
      wave_sync();
      if (lane < nread && start < take) mark[start] = lane;
      wave_sync();
      const int ei = wave_inclusive_max(mark[lane]);
      const int e_start = __shfl(start, ei < 0 ? 0 : ei, kWave);
      const int e_first = __shfl(e.x, ei < 0 ? 0 : ei, kWave);
      if (kfull < nread) {
        const int pstart = __shfl(start, kfull, kWave);
        if (pstart < take && lane == kfull)
          stk[sp - 1 - kfull] = make_int2(e.x + (take - pstart), e.y - (take - pstart));
      }
      sp -= kfull;
      const int node = e_first + (lane - e_start);
      if (__ballot(lane < take && (node < 0 || node >= nslots))) {
        if (lane == 0) atomicOr(&a.info->err, kErrStack);
        break;
      }
      bool taken = false;
      int mass = 0;
      if (lane < take) {
        const NodeRec r = a.nodes[node];
        double d2 = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double ek = fmax(0.0, fmax(elo[k] - r.com[k], r.com[k] - ehi[k]));
          d2 += ek * ek;
        }
        if (r.child < 0) {
          is_cand = !RUNS && r.count > 0 && d2 <= rad * rad;  // a particle within rad of the box
          taken = RUNS && r.count > 0 && (!SLICES || (r.first >= p0 && r.first < p1));
          j = r.first;
          px = r.com[0];
          py = r.com[1];
          pz = r.com[2];
          pm = r.m;
        } else {
          // every particle of the cell lies within R of its centre of mass
          const double R = (kHalfSqrt3 * r.l + r.s) * (1.0 + 1e-9) + rad;
          push = !(d2 > R * R);
          if (SLICES) push = push && r.first < p1 && r.first + r.count > p0;
          if (RUNS && !SLICES) {
            const double in = rad - (R - rad);
            mass = push && r.count > kNbRun && in > 0.0 && d2 <= in * in ? r.count : 0;
          }
          taken = RUNS && push && r.count <= kNbRun;
          push = push && !taken;
          rng = make_int2(r.child, r.nchild);
        }
        if (RUNS && taken) {
          tf = SLICES ? max(r.first, p0) : r.first;
          te = SLICES ? min(r.first + r.count, p1) : r.first + r.count;
        }
      }
      if (RUNS) {
        const unsigned long long tm = __ballot(taken);
        const int before = __shfl_up(te, 1, kWave);
        const bool on = lane > 0 && taken && ((tm >> (lane - 1)) & 1ull) && before == tf;
        inner = __ballot(on);
        heads = tm & ~inner;
        if (!SLICES && __ballot(mass != 0)) {
          inside += __builtin_amdgcn_readlane(wave_inclusive_sum(mass), kWave - 1);
          outlier = inside >= a.out_min;
          if (outlier) break;
        }
      }
      }
      const unsigned long long pmask = __ballot(push), cm = __ballot(is_cand);
      const int npush = __popcll(pmask), nc = __popcll(cm);
      wave_sync();
      if (sp + npush > kNbStack) {
        if (lane == 0) atomicOr(&a.info->err, kErrStack);
        break;
      }
      if (push) stk[sp + rank_below(pmask)] = rng;
      if (is_cand) {
        const int q = ncand + rank_below(cm);
        cd.c[q] = CandRec{px, py, pz, pm};
        const double qx = (px - cen[0]) * sc, qy = (py - cen[1]) * sc, qz = (pz - cen[2]) * sc;
        cd.f[q] = make_float4(-2.0f * (float)qx, -2.0f * (float)qy, -2.0f * (float)qz,
                              (float)(qx * qx + qy * qy + qz * qz));
        cd.j[q] = j;
      }
      sp += npush;
      ncand += nc;
      wave_sync();
      if (ncand >= kWave) {
        flush<kNbBlocks, RHO, !RUNS>(a, cd, mark, kWave, gf, gc, nb, lane, fb, ft, hb, cb, rb, ob, lb, plain, tests);
        // the rest (at most 64) move to the front
        ncand -= kWave;
        wave_sync();
        if (lane < ncand) {
          cd.c[lane] = cd.c[kWave + lane];
          cd.f[lane] = cd.f[kWave + lane];
          cd.j[lane] = cd.j[kWave + lane];
        }
        wave_sync();
      }
    }
    if (RUNS && outlier) {
      if (lane == 0) a.out[atomicAdd(&a.info->nb_out, 1)] = g;
      wave_sync();
      continue;
    }
    flush<kNbBlocks, RHO, !RUNS>(a, cd, mark, ncand, gf, gc, nb, lane, fb, ft, hb, cb, rb, ob, lb, plain, tests);
    all_tests += (unsigned long long)tests;
    wave_sync();
    if (SLICES && parts > 1) {
#pragma unroll
      for (int b = 0; b < kNbBlocks; ++b) {
        const int u = b * kWave + lane;
        if (b < nb && u < gc) {
          const int64_t at = (int64_t)unit * a.n_crit + u;
          a.part_count[at] = cb[b];
          a.part_rho[at] = rb[b];
          pairs += (unsigned long long)cb[b];
        }
      }
      continue;
    }
    // outputs in input order
    bool short_list = false;
#pragma unroll
    for (int b = 0; b < kNbBlocks; ++b) {
      const int i = gf + b * kWave + lane;
      if (b < nb && i < gf + gc) {
        const int o = a.perm[i];
        if (a.count) a.count[o] = cb[b];
        if (RHO) a.rho[o] = __dadd_rn(__dmul_rn(a.smass[i], sph_sigma(hb[b])), rb[b]);
        if (!RUNS && (int64_t)cb[b] != lb[b]) short_list = true;
        pairs += (unsigned long long)cb[b];
      }
    }
    if (__ballot(short_list) && lane == 0) atomicOr(&a.info->err, kErrListSpace);
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    pairs += __shfl_xor(pairs, d, kWave);
    all_tests += __shfl_xor(all_tests, d, kWave);
  }
  if (lane == 0 && (pairs || all_tests)) {
    atomicAdd(&a.info->nb_pairs, pairs);
    atomicAdd(&a.info->nb_tests, all_tests);
  }
}

// An outlier's members: its parts in order.
__global__ __launch_bounds__(256) void k_nb_parts(NeighborArgs a) {
  const int nout = a.info->nb_out, per = slices_per_outlier(nout);
  for (int o = blockIdx.x; o < nout; o += gridDim.x) {
    const int g = a.out[o];
    const int gf = a.ginfo[3 * g], gc = a.ginfo[3 * g + 1], gs = a.ginfo[3 * g + 2];
    const int parts = slices_of(per, a.sys[gs].count), u = threadIdx.x;
    if (parts < 2 || u >= gc) continue;
    int c = 0;
    double r = 0.0;
#pragma unroll 4
    for (int k = 0; k < parts; ++k) {
      const int64_t at = ((int64_t)o * per + k) * a.n_crit + u;
      c += a.part_count[at];
      r = __dadd_rn(r, a.part_rho[at]);
    }
    const int i = gf + u, to = a.perm[i];
    if (a.count) a.count[to] = c;
    if (a.rho) a.rho[to] = __dadd_rn(__dmul_rn(a.smass[i], sph_sigma(a.h[to])), r);
  }
}

}  // namespace

template <bool RUNS, bool SLICES, bool RHO>
static auto kernel(int n_crit) {
  return n_crit <= kWave ? k_neighbors<1, RUNS, SLICES, RHO>
                         : (n_crit <= 2 * kWave ? k_neighbors<2, RUNS, SLICES, RHO>
                                                : k_neighbors<BH_MAX_NCRIT / kWave, RUNS, SLICES, RHO>);
}
template <bool RUNS, bool SLICES>
static auto kernel(int n_crit, bool rho) {
  return rho ? kernel<RUNS, SLICES, true>(n_crit) : kernel<RUNS, SLICES, false>(n_crit);
}

template <bool RUNS, bool SLICES>
static int blocks_per_cu(int n_crit, bool rho) {
  int b = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kernel<RUNS, SLICES>(n_crit, rho), kWave, 0);
  return e != hipSuccess || b < 1 ? 8 : b;
}

int neighbors_blocks_per_cu(int n_crit, bool lists, bool rho) {
  return lists ? blocks_per_cu<false, false>(n_crit, rho)
               : std::min(blocks_per_cu<true, false>(n_crit, rho), blocks_per_cu<true, true>(n_crit, rho));
}

template <bool RUNS, bool SLICES>
static void launch(const NeighborArgs &a, int grid, hipStream_t s) {
  kernel<RUNS, SLICES>(a.n_crit, a.rho != nullptr)<<<(unsigned)grid, kWave, 0, s>>>(a);
}

int neighbors_out_min(int64_t n) {
  return n <= 2 * kNbOutMin ? INT32_MAX : (int)std::max<int64_t>(n / 16, kNbOutMin);
}
size_t neighbors_parts(int n_crit) { return (size_t)kNbRows * (size_t)n_crit; }

void neighbors_device(const NeighborArgs &a, int grid, hipStream_t s) {
  k_nb_reset<<<1, 64, 0, s>>>(a.info);
  if (a.nbr) {
    launch<false, false>(a, grid, s);
    return;
  }
  launch<true, false>(a, grid, s);
  if (a.out) {
    launch<true, true>(a, grid, s);
    k_nb_parts<<<256, 256, 0, s>>>(a);
  }
}

}  // namespace bh
