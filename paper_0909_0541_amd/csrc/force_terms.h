// One list entry's terms of Eq. (1) in FP32, shared by the force kernels
// (k_force.hip: entries from scalar loads; k_wide.hip: entries from LDS).
#pragma once

#include "bh_device.h"

namespace bh {

struct Member {
  float x, y, z;     // FP32 x_i - c_g
  float lx, ly, lz;  // rounding residue of x_i - c_g
  float ax, ay, az, pt;
  double dx, dy, dz, dp;
};

__device__ __forceinline__ void member_init(Member &M, double rx, double ry, double rz) {
  M.x = (float)rx;
  M.y = (float)ry;
  M.z = (float)rz;
  M.lx = (float)__dsub_rn(rx, (double)M.x);
  M.ly = (float)__dsub_rn(ry, (double)M.y);
  M.lz = (float)__dsub_rn(rz, (double)M.z);
  M.ax = M.ay = M.az = M.pt = 0.0f;
  M.dx = M.dy = M.dz = M.dp = 0.0;
}

// Potential of a member's own entry (dx = 0 exactly), as the sums add it.
__device__ __forceinline__ double self_potential(double mass, float eps2) {
  return (double)((float)mass * __builtin_amdgcn_rsqf(__builtin_fmaf(0.0f, 0.0f, eps2)));
}

// The quadrupole term of one cell entry at relative position (dx, dy, dz),
// with R^2 = |u|^2 + eps^2 and ri = 1/R; a = 3 (xx, yy, zz, xy), b = (3 xz,
// 3 yz, T, 1.5 T).  With S3 = 3 S and w = u.S3.u the terms above read
//   force       r5 (2.5 w ri^2 - 1.5 T) u - r5 S3 u
//   -potential  0.5 r5 (w - T R^2),        r5 = ri^5.
__device__ __forceinline__ void quad_term(Member &M, const float4 a, const float4 b, float dx, float dy, float dz,
                                          float R2, float ri) {
  const float sx = __builtin_fmaf(a.x, dx, __builtin_fmaf(a.w, dy, b.x * dz));
  const float sy = __builtin_fmaf(a.w, dx, __builtin_fmaf(a.y, dy, b.y * dz));
  const float sz = __builtin_fmaf(b.x, dx, __builtin_fmaf(b.y, dy, a.z * dz));
  const float w = __builtin_fmaf(dx, sx, __builtin_fmaf(dy, sy, dz * sz));
  const float ri2 = ri * ri;
  const float r5 = ri2 * ri2 * ri;
  const float c = r5 * __builtin_fmaf(2.5f * w, ri2, -b.w);
  M.ax = __builtin_fmaf(-r5, sx, __builtin_fmaf(c, dx, M.ax));
  M.ay = __builtin_fmaf(-r5, sy, __builtin_fmaf(c, dy, M.ay));
  M.az = __builtin_fmaf(-r5, sz, __builtin_fmaf(c, dz, M.az));
  M.pt = __builtin_fmaf(0.5f * r5, __builtin_fmaf(-b.z, R2, w), M.pt);
}

// U entries (value e, rounding residue l when NEAR) against this lane's
// member, written stage by stage across the U independent terms.  With QUAD,
// cell[u] says whether entry u is a cell, qa and qb its packed moments.
template <int U, bool NEAR, bool QUAD>
__device__ __forceinline__ void entry_terms(Member &M, const float4 (&e)[U], const float4 (&l)[U], float eps2,
                                            const bool (&cell)[U], const float4 (&qa)[U], const float4 (&qb)[U]) {
  float dx[U], dy[U], dz[U], q[U], mr[U], ri[U], R2[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    dx[u] = e[u].x - M.x;
    dy[u] = e[u].y - M.y;
    dz[u] = e[u].z - M.z;
  }
  if (NEAR) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      dx[u] += l[u].x - M.lx;
      dy[u] += l[u].y - M.ly;
      dz[u] += l[u].z - M.lz;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) q[u] = __builtin_fmaf(dx[u], dx[u], eps2);
#pragma unroll
  for (int u = 0; u < U; ++u) q[u] = __builtin_fmaf(dy[u], dy[u], q[u]);
#pragma unroll
  for (int u = 0; u < U; ++u) q[u] = __builtin_fmaf(dz[u], dz[u], q[u]);
  if (QUAD) {
#pragma unroll
    for (int u = 0; u < U; ++u) R2[u] = q[u];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) q[u] = __builtin_amdgcn_rsqf(q[u]);  // 1/r
  if (QUAD) {
#pragma unroll
    for (int u = 0; u < U; ++u) ri[u] = q[u];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    mr[u] = e[u].w * q[u];
    q[u] = q[u] * q[u];  // 1/r^2
  }
#pragma unroll
  for (int u = 0; u < U; ++u) q[u] = mr[u] * q[u];  // m/r^3
#pragma unroll
  for (int u = 0; u < U; ++u) {
    M.ax = __builtin_fmaf(q[u], dx[u], M.ax);
    M.ay = __builtin_fmaf(q[u], dy[u], M.ay);
    M.az = __builtin_fmaf(q[u], dz[u], M.az);
    M.pt += mr[u];
  }
  if (QUAD) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (cell[u]) quad_term(M, qa[u], qb[u], dx[u], dy[u], dz[u], R2[u], ri[u]);
  }
}

__device__ __forceinline__ void fold(Member &M) {
  M.dx += (double)M.ax;
  M.dy += (double)M.ay;
  M.dz += (double)M.az;
  M.dp += (double)M.pt;
  M.ax = M.ay = M.az = M.pt = 0.0f;
}

// A stage of entries [lo, hi) in LDS against this lane's member: all of them
// (R = 1, read as broadcasts), or with R lane partitions those of partition
// sub.  qs: the entries' packed moments and cell: node slots (-1 a particle).
// U entries' terms at a time: with QUAD the order in which they are added.
template <bool NEAR, bool QUAD, int U = QUAD ? 2 : 4>
__device__ __forceinline__ void stage_sum(Member &M, const float4 *e, const float4 *l, const int32_t *slot,
                                          const float4 *qs, int lo, int hi, int sub, int R, float eps2) {
  int k = lo + sub;
  for (; k + (U - 1) * R < hi; k += U * R) {
    float4 ev[U], lv[U], qa[U], qb[U];
    bool cell[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = k + u * R;
      ev[u] = e[j];
      lv[u] = NEAR ? l[j] : ev[u];
      cell[u] = QUAD && slot[j] >= 0;
      qa[u] = QUAD ? qs[2 * j] : ev[u];
      qb[u] = QUAD ? qs[2 * j + 1] : ev[u];
    }
    entry_terms<U, NEAR, QUAD>(M, ev, lv, eps2, cell, qa, qb);
  }
  for (; k < hi; k += R) {
    const float4 ev[1] = {e[k]}, lv[1] = {NEAR ? l[k] : e[k]};
    const bool cell[1] = {QUAD && slot[k] >= 0};
    const float4 qa[1] = {QUAD ? qs[2 * k] : ev[0]}, qb[1] = {QUAD ? qs[2 * k + 1] : ev[0]};
    entry_terms<1, NEAR, QUAD>(M, ev, lv, eps2, cell, qa, qb);
  }
}

}  // namespace bh
