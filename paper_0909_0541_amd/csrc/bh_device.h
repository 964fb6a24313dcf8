// Device-side helpers shared by the kernels of libbh (wave64, gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bh_internal.h"

namespace bh {

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// One value per wavefront from an atomic counter: every lane executes the
// atomic (lane 0 adds one, the others zero) so that no divergent branch
// precedes the broadcast of lane 0's result.  Call with all lanes active and
// a counter address the compiler can see is the same on every lane (derive
// a computed index with readfirstlane): only then is the atomic issued as
// one request; 64 requests on one counter serialise behind each other, which
// once made the walk ten times slower.
__device__ __forceinline__ int take_one(int *counter, int lane) {
  const int t = atomicAdd(counter, lane == 0 ? 1 : 0);
  return __builtin_amdgcn_readfirstlane(t);
}

// Number of set bits of m below this lane.
__device__ __forceinline__ int rank_below(unsigned long long m) {
  return (int)__popcll(m & __lanemask_lt());
}

// Inclusive prefix sum and maximum over the 64 lanes of a wave, in data-
// parallel-primitive (DPP) moves between lanes instead of LDS permutes:
// shifts by 1, 2, 4 and 8 lanes within each row of 16 (a Hillis-Steele scan
// of the row), then row 15's last lane broadcast into rows 1 and 3 and lane
// 31 into rows 2 and 3.  Lanes whose source lies outside the row take the
// identity.  Call with all lanes active.
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;

__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr1, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr2, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr4, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr8, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowBcast15, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowBcast31, 0xc, 0xf, false);
  return v;
}

// The same within each row of 16 lanes.
__device__ __forceinline__ int wave_row_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr1, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr2, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppRowShr4, 0xf, 0xf, false);
  return v + __builtin_amdgcn_update_dpp(0, v, kDppRowShr8, 0xf, 0xf, false);
}

__device__ __forceinline__ int wave_inclusive_max(int v) {
  constexpr int kId = -2147483647 - 1;
  v = max(v, __builtin_amdgcn_update_dpp(kId, v, kDppRowShr1, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(kId, v, kDppRowShr2, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(kId, v, kDppRowShr4, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(kId, v, kDppRowShr8, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(kId, v, kDppRowBcast15, 0xa, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(kId, v, kDppRowBcast31, 0xc, 0xf, false));
  return v;
}

__device__ __forceinline__ double shfl_xor_d(double v, int mask) {
  int2 a = *reinterpret_cast<int2 *>(&v);
  a.x = __shfl_xor(a.x, mask, kWave);
  a.y = __shfl_xor(a.y, mask, kWave);
  return *reinterpret_cast<double *>(&a);
}

__device__ __forceinline__ double shfl_d(double v, int lane) {
  int2 a = *reinterpret_cast<int2 *>(&v);
  a.x = __shfl(a.x, lane, kWave);
  a.y = __shfl(a.y, lane, kWave);
  return *reinterpret_cast<double *>(&a);
}

__device__ __forceinline__ int64_t shfl_i64(int64_t v, int lane) {
  const int lo = __shfl((int)(uint32_t)v, lane, kWave), hi = __shfl((int)(v >> 32), lane, kWave);
  return ((int64_t)hi << 32) | (uint32_t)lo;
}

// Node tests after which a group's walk is an outlier's: four times what such
// a group takes in an ordinary place, at least out_min.  Lists hold about
// (60 + 25 sqrt(n_crit)) theta^-1.5 entries per factor of eight in particle
// number (mean lists of clustered boxes, Plummer and uniform spheres from
// 30,000 to 4 million particles at theta 0.33 to 0.75 lie within 0.6 to 1.4
// of that), and a walk tests 1.3 nodes an entry.  A function of the group
// alone, so that the same groups are outliers in every run.  Systems of up to
// out_tree particles have none.
__device__ __forceinline__ int outlier_cap(int out_min, int out_tree, int n_crit, int count, double theta) {
  if (out_min <= 0 || count <= out_tree || !(theta > 0.0)) return 0;
  const float octaves = fmaxf(1.0f, log2f((float)count / (float)n_crit) * (1.0f / 3.0f));
  const float th = (float)theta;
  const float cap = 5.2f * (60.0f + 25.0f * sqrtf((float)n_crit)) * octaves / (th * sqrtf(th));
  return max(out_min, (int)fminf(cap, 1e9f));
}

// Place among the outliers; beyond the last one an error that makes the host
// walk every group whole.  One lane.
__device__ __forceinline__ int take_outlier(DevInfo *info, int places) {
  const int o = atomicAdd(&info->n_out, 1);
  if (o < places) return o;
  atomicOr(&info->err, kErrWide);
  return -1;
}

// Octal digits shared by two 63-bit keys (21 when equal).
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
  uint64_t x = a ^ b;
  if (x == 0) return kKeyLevels;
  int hb = 63 - __clzll((long long)x);
  return 20 - hb / 3;
}

// Octant (0..7) of a key at level l (1..21).
__device__ __forceinline__ int key_digit(uint64_t k, int l) {
  return (int)((k >> (3 * (kKeyLevels - l))) & 7u);
}

// Shift that keeps the first l octal digits of a key.
__device__ __forceinline__ int prefix_shift(int l) { return 3 * (kKeyLevels - l); }

// First index in [lo, hi) whose key prefix (k >> sh) is >= p (keys sorted).
__device__ __forceinline__ int lower_bound_prefix(const uint64_t *__restrict__ keys, int lo, int hi, uint64_t p,
                                                  int sh) {
  while (lo < hi) {
    int mid = lo + ((hi - lo) >> 1);
    if ((keys[mid] >> sh) < p) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// First index in [lo, hi) whose key prefix is > p.
__device__ __forceinline__ int upper_bound_prefix(const uint64_t *__restrict__ keys, int lo, int hi, uint64_t p,
                                                  int sh) {
  while (lo < hi) {
    int mid = lo + ((hi - lo) >> 1);
    if ((keys[mid] >> sh) <= p) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Galloping searches around a known position j whose key prefix equals p:
// steps of 1, 2, 4, ... away from j, then a binary search in the last step,
// so that small cells cost a few cached loads instead of a search over the
// whole system.
// First index in [lo, j] whose prefix equals p.
__device__ __forceinline__ int gallop_first(const uint64_t *__restrict__ keys, int lo, int j, uint64_t p, int sh) {
  int good = j, bad = lo - 1;
  for (int step = 1;; step <<= 1) {
    const int probe = good - step;
    if (probe < lo) break;
    if ((keys[probe] >> sh) < p) {
      bad = probe;
      break;
    }
    good = probe;
  }
  return lower_bound_prefix(keys, bad + 1, good, p, sh);
}

// First index in (j, hi) whose prefix exceeds p (hi if none).
__device__ __forceinline__ int gallop_past(const uint64_t *__restrict__ keys, int j, int hi, uint64_t p, int sh) {
  int good = j, bad = hi;
  for (int step = 1;; step <<= 1) {
    const int probe = good + step;
    if (probe >= hi) break;
    if ((keys[probe] >> sh) > p) {
      bad = probe;
      break;
    }
    good = probe;
  }
  return upper_bound_prefix(keys, good + 1, bad, p, sh);
}

// System owning Morton position j (systems occupy consecutive ranges).
__device__ __forceinline__ int system_of(const SysInfo *__restrict__ sys, int nsys, int j) {
  int lo = 0, hi = nsys - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (sys[mid].first <= j) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Cell coordinate (21 bits) of a position along one axis.
__device__ __forceinline__ uint32_t quantise(double x, double lo, double scale) {
  double u = __dsub_rn(x, lo);
  u = __dmul_rn(u, scale);
  if (!(u >= 0.0)) return 0u;
  if (u >= (double)kQMax) return kQMax;
  return (uint32_t)u;  // truncation == floor for u >= 0
}

}  // namespace bh
