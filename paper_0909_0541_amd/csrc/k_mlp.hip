// Per-group opening angle chosen by a small network (12 -> 64 -> 64 -> 1).
//
// The paper uses one theta for every particle and studies how it trades
// accuracy for work (Sec. 3.5, Table "theta").  Here each group gets its own theta from 12
// features that describe how it sits in the surrounding mass (c members,
// c_g box centre, R box half-diagonal, x_g and m_g the members' centre of mass
// and mass, A1 the smallest cell with at least two sub-cells (not a bucket)
// that holds more than c particles, A2 the next such cell above it, A1 again
// at the root):
//   f0 = log2 c, f1 = log2(1 + R/eps), f2 = |x_g - c_g| / (R + eps),
//   f3 = log2(l(A1) / (R + eps)), f4 = log2(m(A1) / m_g),
//   f5 = |com(A1) - c_g| / l(A1), f11 = log2(m(A2) / m_g),
// and, from the group's interaction list at theta = 1 (the probe walk) with
// d = com - c_g over the entries outside the box (the probe walk, one wave per
// group, computes all twelve):
//   f6 = log2(|sum m d / (d^2 + eps^2)^1.5| + 2^-100),
//   f7 = log2(sum m / (d^2 + eps^2) + 2^-100),
//   f8 = log2(1 + single particles outside the box), f9 = log2(list length),
//   f10 = log2(mass of the entries inside the box / m_g); then
//   theta = 0.3 + 0.7 sigmoid(w3 . tanh(W2 tanh(W1 x' + b1) + b2) + b3 + shift),
// x' = (x - mu) / sigma.  Inference runs on the matrix cores in bfloat16
// (v_mfma_f32_16x16x16_bf16, FP32 accumulation); training runs in FP32 (the
// forward and backward products on the FP32 matrix instructions), gradients
// summed over the batch in a fixed order.
//
// Parameters: one FP32 vector W1 [64][12], b1 [64], W2 [64][64], b2 [64],
// w3 [64], b3 [1].
#include <algorithm>

#include "bh_device.h"

namespace bh {

namespace {

constexpr int kIn = 12, kHid = 64;
constexpr int oW1 = 0, oB1 = oW1 + kHid * kIn, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid, oW3 = oB2 + kHid,
              oB3 = oW3 + kHid;
static_assert(oB3 + 1 == kMlpParams, "parameter layout");

// ---- inference (bfloat16 matrix cores) --------------------------------------

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> bfloat16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ short to_bf16(float x) {
  const uint32_t u = __float_as_uint(x);
  return (short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float sigmoid_theta(float y) {
  return kThetaMin + kThetaSpan / (1.0f + expf(-y));
}

// One wave per tile of 16 rows.  Operand layout of the 16x16x16 product
// (wave64): lane l holds A[l % 16][4 (l / 16) + v] and B[4 (l / 16) + v][l % 16]
// for v = 0..3, and the result D[4 (l / 16) + v][l % 16].
__global__ __launch_bounds__(kWave) void k_mlp_infer(const float *__restrict__ P, const float *__restrict__ mu,
                                                     const float *__restrict__ sigma, const float *__restrict__ x,
                                                     int64_t rows_host, const DevInfo *__restrict__ info, float shift,
                                                     float *__restrict__ theta) {
  __shared__ short h1[16][kHid + 4];
  const int lane = lane_id();
  const int col = lane & 15, kb = lane >> 4;
  const int64_t rows = rows_host >= 0 ? rows_host : (int64_t)info->n_groups;
  const int64_t tiles = (rows + 15) / 16;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t row = t * 16 + col;
    bf16x4 ax;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = 4 * kb + v;
      float xv = 0.0f;
      if (k < kIn && row < rows) xv = (x[row * kIn + k] - mu[k]) / sigma[k];
      ax[v] = (k < kIn) ? to_bf16(xv) : (short)0;
    }
    // layer 1: 4 column blocks of 16 hidden units
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const int j = 16 * nb + col;
      bf16x4 bw;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = 4 * kb + v;
        bw[v] = (k < kIn) ? to_bf16(P[oW1 + j * kIn + k]) : (short)0;
      }
      f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
      z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ax, bw, z, 0, 0, 0);
      const float b = P[oB1 + j];
#pragma unroll
      for (int v = 0; v < 4; ++v) h1[4 * kb + v][j] = to_bf16(tanhf(z[v] + b));
    }
    __syncthreads();
    // layer 2 and the output layer
    float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const int j = 16 * nb + col;
      f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        bf16x4 ah, bw;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = 16 * ks + 4 * kb + v;
          ah[v] = h1[col][k];
          bw[v] = to_bf16(P[oW2 + j * kHid + k]);
        }
        z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bw, z, 0, 0, 0);
      }
      const float b = P[oB2 + j], w = P[oW3 + j];
#pragma unroll
      for (int v = 0; v < 4; ++v) part[v] += w * tanhf(z[v] + b);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) part[v] += __shfl_xor(part[v], d, kWave);
    }
    if (col == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = t * 16 + 4 * kb + v;
        if (r < rows) theta[r] = sigmoid_theta(part[v] + P[oB3] + shift);
      }
    }
    __syncthreads();
  }
}

// ---- training (FP32) ----------------------------------------------------------

// Forward, backward and the batch's parameter gradient on the matrix cores
// in FP32 (16x16x4 products, FP32 operands and accumulation).  Operand layout
// (wave64): lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and of the
// result D[4 (l / 16) + v][l % 16] for v = 0..3.
//
// A block takes tiles of 16 samples; its four waves each own 16 hidden units
// of both layers (forward and both deltas) and the gradient rows of those
// units, summed over the block's tiles in registers.  The tile's activations
// and deltas pass between the waves through LDS.  What bounds it is the chain
// of one tile (loads, four small products, three barriers), not the flops, so
// tiles go one to a block (up to kTrainBlocks blocks, then several to a
// block), and a block writes one partial gradient; k_mlp_reduce adds the
// partials in block order.  Batch 1024: 364 us for a gradient and an Adam step
// with one thread a sample and one thread a parameter's serial sum over the
// batch, 20 us like this.
constexpr int kTrainBlocks = 256;
constexpr int kTrainTile = 16;
constexpr int kPartRow = (kMlpParams + 1 + 63) / 64 * 64;  // parameters, then the loss

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(256) void k_mlp_train(const float *__restrict__ P, const float *__restrict__ mu,
                                                   const float *__restrict__ sigma, const float *__restrict__ x,
                                                   const float *__restrict__ target, const float *__restrict__ w,
                                                   int B, float *__restrict__ part) {
  constexpr int kPad = kHid + 1;
  __shared__ float W2[kHid][kPad], W1[kHid][kTrainTile + 1];
  __shared__ float xn[kTrainTile][kTrainTile + 1], h1[kTrainTile][kPad], h2[kTrainTile][kPad];
  __shared__ float dz1[kTrainTile][kPad], dz2[kTrainTile][kPad];
  __shared__ float dys[kTrainTile], ls[kTrainTile], red[256];
  const int t = threadIdx.x, lane = lane_id(), wv = t / kWave;
  const int col = lane & 15, q = lane >> 4;
  // sum of the sample weights (every block the same way)
  float wacc = 0.0f;
#pragma unroll 8
  for (int b = t; b < B; b += 256) wacc += w[b];
  red[t] = wacc;
  for (int e = t; e < kHid * kHid; e += 256) W2[e / kHid][e % kHid] = P[oW2 + e];
  for (int e = t; e < kHid * kTrainTile; e += 256) {
    const int j = e / kTrainTile, k = e % kTrainTile;
    W1[j][k] = k < kIn ? P[oW1 + j * kIn + k] : 0.0f;
  }
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) red[t] += red[t + h];
    __syncthreads();
  }
  const float W = red[0];
  const int j0 = 16 * wv;  // this wave's hidden units
  const float bias1 = P[oB1 + j0 + col], bias2 = P[oB2 + j0 + col], w3 = P[oW3 + j0 + col];
  f32x4 g2[4], g1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) g2[nb] = g1;
  float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, loss = 0.0f;  // (threads 0..63: one hidden unit each)
  const int tiles = (B + kTrainTile - 1) / kTrainTile;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int b0 = tile * kTrainTile;
    {
      const int s = t / kTrainTile, k = t % kTrainTile;
      xn[s][k] = (k < kIn && b0 + s < B) ? (x[(int64_t)(b0 + s) * kIn + k] - mu[k]) / sigma[k] : 0.0f;
    }
    __syncthreads();
    f32x4 z = {bias1, bias1, bias1, bias1};
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) z = mfma4(xn[col][4 * ks + q], W1[j0 + col][4 * ks + q], z);
    float a1[4], a2[4];  // this lane's activations: samples 4 q + v, unit j0 + col
#pragma unroll
    for (int v = 0; v < 4; ++v) h1[4 * q + v][j0 + col] = a1[v] = tanhf(z[v]);
    __syncthreads();
    z = f32x4{bias2, bias2, bias2, bias2};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) z = mfma4(h1[col][4 * ks + q], W2[j0 + col][4 * ks + q], z);
#pragma unroll
    for (int v = 0; v < 4; ++v) h2[4 * q + v][j0 + col] = a2[v] = tanhf(z[v]);
    __syncthreads();
    {
      // the outputs of samples 4 wv + q, sixteen lanes a sample
      const int s = 4 * wv + q;
      float y = 0.0f;
#pragma unroll
      for (int u = 0; u < 4; ++u) y += P[oW3 + 16 * u + col] * h2[s][16 * u + col];
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) y += __shfl_xor(y, d, kWave);
      y += P[oB3];
      if (col == 0) {
        const int b = b0 + s;
        float dy = 0.0f, l = 0.0f;
        if (b < B) {
          const float sg = 1.0f / (1.0f + expf(-y));
          const float r = kThetaMin + kThetaSpan * sg - target[b];
          const float wb = w[b];
          l = wb * r * r / W;
          dy = (2.0f * wb * r / W) * kThetaSpan * sg * (1.0f - sg);
        }
        dys[s] = dy;
        ls[s] = l;
      }
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) dz2[4 * q + v][j0 + col] = dys[4 * q + v] * w3 * (1.0f - a2[v] * a2[v]);
    __syncthreads();
    z = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) z = mfma4(dz2[col][4 * ks + q], W2[4 * ks + q][j0 + col], z);
#pragma unroll
    for (int v = 0; v < 4; ++v) dz1[4 * q + v][j0 + col] = z[v] * (1.0f - a1[v] * a1[v]);
    // gradient rows j0 .. j0 + 15: sums over the tile's samples
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const float a = dz2[4 * ks + q][j0 + col];
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) g2[nb] = mfma4(a, h1[4 * ks + q][16 * nb + col], g2[nb]);
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) g1 = mfma4(dz1[4 * ks + q][j0 + col], xn[4 * ks + q][col], g1);
    if (t < kHid) {
      float s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
#pragma unroll
      for (int s = 0; s < kTrainTile; ++s) {
        s1 += dz1[s][t];
        s2 += dz2[s][t];
        s3 += dys[s] * h2[s][t];
      }
      gb1 += s1;
      gb2 += s2;
      gw3 += s3;
    }
    if (t == kHid) {
      float s4 = 0.0f, s5 = 0.0f;
      for (int s = 0; s < kTrainTile; ++s) {
        s4 += dys[s];
        s5 += ls[s];
      }
      gb3 += s4;
      loss += s5;
    }
    __syncthreads();
  }
  float *o = part + (int64_t)blockIdx.x * kPartRow;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int j = j0 + 4 * q + v;
    if (col < kIn) o[oW1 + j * kIn + col] = g1[v];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) o[oW2 + j * kHid + 16 * nb + col] = g2[nb][v];
  }
  if (t < kHid) {
    o[oB1 + t] = gb1;
    o[oB2 + t] = gb2;
    o[oW3 + t] = gw3;
  }
  if (t == kHid) {
    o[oB3] = gb3;
    o[kMlpParams] = loss;
  }
}

// The blocks' partial gradients added in block order, in four runs of blocks
// (one per wave) whose sums are added in order.
__global__ __launch_bounds__(256) void k_mlp_reduce(const float *__restrict__ part, int nblocks,
                                                    float *__restrict__ grad, float *__restrict__ loss) {
  __shared__ float red[4][kWave];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int p = blockIdx.x * kWave + lane;  // p < kPartRow
  const int per = (nblocks + 3) / 4;
  const int lo = min(wv * per, nblocks), hi = min(lo + per, nblocks);
  float s = 0.0f;
  if (p <= kMlpParams)
#pragma unroll 16
    for (int b = lo; b < hi; ++b) s += part[(int64_t)b * kPartRow + p];
  red[wv][lane] = s;
  __syncthreads();
  if (wv != 0) return;
  s = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
  if (p < kMlpParams) grad[p] = s;
  else if (p == kMlpParams && loss) *loss = s;
}

__global__ void k_adam(float *__restrict__ P, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  P[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace


void mlp_infer_device(const float *params, const float *mu, const float *sigma, const float *x, int64_t rows,
                      int64_t cap_rows, const DevInfo *info, float shift, float *theta, hipStream_t s) {
  const int64_t tiles = (cap_rows + 15) / 16;
  if (tiles <= 0) return;
  const unsigned grid = (unsigned)std::min<int64_t>(tiles, 4096);
  k_mlp_infer<<<grid, kWave, 0, s>>>(params, mu, sigma, x, rows, info, shift, theta);
}

static int train_blocks(int B) { return std::min((B + kTrainTile - 1) / kTrainTile, kTrainBlocks); }

size_t mlp_part_bytes(int B) { return sizeof(float) * (size_t)train_blocks(B) * kPartRow; }

void mlp_grad_device(const float *params, const float *mu, const float *sigma, int B, const float *x,
                     const float *target, const float *w, float *part, float *grad, float *loss, hipStream_t s) {
  const int blocks = train_blocks(B);
  k_mlp_train<<<(unsigned)blocks, 256, 0, s>>>(params, mu, sigma, x, target, w, B, part);
  k_mlp_reduce<<<(unsigned)(kPartRow / kWave), 256, 0, s>>>(part, blocks, grad, loss);
}

void adam_device(float *params, const float *grad, float *m, float *v, int n, float lr, float b1, float b2, float eps,
                 int step, hipStream_t s) {
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  k_adam<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(params, grad, m, v, n, lr, b1, b2, eps, c1, c2);
}

}  // namespace bh
