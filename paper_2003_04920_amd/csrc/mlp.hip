// The learned sampling proposal's network on the device: features (sample
// coordinates + obstacle encoding, zero-padded to K = 288) -> 256 -> 256 -> 1 logit,
// ReLU hidden layers, bfloat16 operands with binary32 accumulation on MFMA, binary32
// master parameters, BCE-with-logits loss, Adam (Kingma and Ba, 2015).
//
// Rounding points (the contract the oracle states): X = bf16(f); A1 = bf16(relu(Z1));
// A2 = bf16(relu(Z2)); weights used by products are bf16 copies of the binary32
// masters; dZ2 = bf16(dz w3^T * [Z2 > 0]); dZ1 = bf16(dZ2 W2^T * [Z1 > 0]).
//
// A sample's whole pass is local to its row, so one kernel (k_net) takes 32 rows from the
// features to the logit and, in training, back to dZ1: eight waves hold the 32 x 256
// activations of a layer, one 32 x 32 block each accumulated by v_mfma_f32_32x32x16_bf16,
// and hand them on in LDS.  Only the weight gradients contract over the batch: k_net leaves
// their operands in fragment order along the batch, k_wgrad multiplies them over splits of
// the batch and k_update adds the splits and the column sums in a fixed order, then takes
// the Adam step.
//
// Bound by: a launch, the chain of a layer's 16 to 18 matrix instructions at one wave each and
// three barriers, not by the matrix cores or memory.  Weights and gradient operands lie in
// the order in which the lanes load them (fragment); by rows, each load touched a line a lane:
// k_net 13.5 and 22.3 us, k_wgrad 16.1, now 8.6, 16.0 and 8.2.  Measured as a call: the
// forward pass of 8,192 rows 48.5 us as five kernels through memory, now 21.8; loss and
// gradients of 4,096 rows 136 us as sixteen, now 37.
#include <string.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "internal.h"
#include "pirrt.h"

using namespace pirrt;

namespace {

constexpr int kIn = 288;      // padded input width (a multiple of 16)
constexpr int kHidden = 256;  // hidden width
constexpr int64_t kOffW1 = 0;
constexpr int64_t kOffB1 = kOffW1 + (int64_t)kIn * kHidden;
constexpr int64_t kOffW2 = kOffB1 + kHidden;
constexpr int64_t kOffB2 = kOffW2 + (int64_t)kHidden * kHidden;
constexpr int64_t kOffW3 = kOffB2 + kHidden;
constexpr int64_t kOffB3 = kOffW3 + kHidden;
constexpr int64_t kNumParams = kOffB3 + 1;
constexpr int kThreads = 256;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even (no NaN reaches here)
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

constexpr int kRows = 32;               // batch rows of a workgroup's tile
constexpr int kNetThreads = 512;        // eight waves, 32 hidden units each
constexpr int kXStride = kIn + 8;       // LDS row strides: 16-byte reads of 16 rows at one
constexpr int kAStride = kHidden + 8;   // column fall into distinct banks
constexpr int kNetGroups = 256;         // workgroups of a training pass at most
constexpr int kSplits = 16;             // batch splits of the weight gradients at most
constexpr int kGradRows = kIn + kHidden;  // rows of gW1 and gW2 together
constexpr int kColSums = 3 * kHidden + 2;  // gb1, gb2, gw3, gb3, loss: per workgroup
static_assert(kHidden == 32 * (kNetThreads / 64), "a wave per 32 hidden units");

// Where element k of feature f lies in an operand that products read along k, in steps of 16:
// the 64 lanes' fragments of one (32 features, step) block follow each other, so that a
// fragment load of a wave is 1 KB in a row (rows 512 bytes apart cost four times the lines).
__device__ __forceinline__ int64_t fragment(int64_t f, int64_t k, int64_t steps) {
  return ((f >> 5) * steps + (k >> 4)) * 512 + ((k >> 3 & 1) * 32 + (f & 31)) * 8 + (k & 7);
}

// What a training pass leaves for the weight gradients: operands in fragment order, the
// batch along k.
struct TrainOut {
  uint16_t* XT;
  uint16_t* A1T;
  uint16_t* dZ1T;
  uint16_t* dZ2T;
  float* colsum;  // [workgroup][kColSums]
  int64_t steps;  // of 16 batch rows
};

// One layer's 32 x 32 block of the wave: K products with 16 at a time, k ascending.  Lane l
// supplies A row l % 32 (LDS) and B column l % 32 (the weights, in fragment order) with the 8
// consecutive k from 8 (l / 32); accumulator register r of lane l holds row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
// The weights' fragments are loaded ahead of the barrier before the layer (Weights), all in
// flight together.
template <int K>
struct Weights {
  bf16x8 b[K / 16];
  __device__ __forceinline__ void load(const uint16_t* w) {
#pragma unroll
    for (int k = 0; k < K / 16; ++k) b[k] = load8(w + 512 * k);
    __builtin_amdgcn_sched_barrier(0);  // issued here, not where they are used
  }
  __device__ __forceinline__ f32x16 product(const uint16_t* a) const {
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
    for (int k = 0; k < K / 16; ++k)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load8(a + 16 * k), b[k], acc, 0, 0, 0);
    return acc;
  }
};

// bf16(relu(z)); in training a unit that is off (z <= 0) is -0, so that its sign carries
// [z > 0] for the backward pass (a zero of either sign adds nothing to a product).
template <bool kTrain>
__device__ __forceinline__ uint16_t activate(float z) {
  return z > 0.0f ? to_bf16(z) : (uint16_t)(kTrain ? 0x8000u : 0u);
}

// Forward pass of rows [32 tile, 32 tile + 32); kTrain: loss, dZ2, dZ1 and the transposed
// operands too.  Without kTrain one tile a workgroup; with it the workgroups loop over the
// tiles and keep their column sums in registers.  Rows past B have zero features and, in
// training, zero dz.
template <bool kTrain>
__global__ void __launch_bounds__(kNetThreads, 2) k_net(int32_t B, int32_t tiles, int32_t in_dim,
                                                        const float* __restrict__ x, const uint16_t* __restrict__ W1t,
                                                        const uint16_t* __restrict__ W2t,
                                                        const uint16_t* __restrict__ W2b,
                                                        const uint16_t* __restrict__ w3b, const float* __restrict__ P,
                                                        const float* __restrict__ y, float* __restrict__ logits,
                                                        TrainOut out) {
  __shared__ __align__(16) uint16_t sx[kRows * kXStride];  // X, then dZ2
  __shared__ __align__(16) uint16_t sa[kRows * kAStride];  // A1
  __shared__ __align__(16) uint16_t sb[kRows * kAStride];  // A2
  __shared__ __align__(16) float w3[kHidden];
  __shared__ float sdz[kRows], sloss[kRows];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const int c = lane & 31, half = lane >> 5;
  const int n = 32 * wave + c;  // the lane's hidden unit
  if (t < kHidden) w3[t] = from_bf16(w3b[t]);
  const float b1 = P[kOffB1 + n], b2 = P[kOffB2 + n], b3 = P[kOffB3];
  float g1 = 0.0f, g2 = 0.0f, g3 = 0.0f, gb3 = 0.0f, gl = 0.0f;  // column sums
  Weights<kIn> w1;
  Weights<kHidden> w2;
  for (int32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t row0 = (int64_t)tile * kRows;
    // (the weights are read again for every tile: kept over the loop they would spill)
    asm volatile("" : "+s"(W1t), "+s"(W2t), "+s"(W2b));
    {  // 16 threads a row, all of a thread's features in flight
      const int r = t / 16, k0 = t % 16;
      const float* xr = x + (row0 + r) * in_dim;
      float f[kIn / 16];
#pragma unroll
      for (int j = 0; j < kIn / 16; ++j) f[j] = row0 + r < B && k0 + 16 * j < in_dim ? xr[k0 + 16 * j] : 0.0f;
      w1.load(W1t + wave * 32 * kIn + 8 * lane);
#pragma unroll
      for (int j = 0; j < kIn / 16; ++j) sx[r * kXStride + k0 + 16 * j] = to_bf16(f[j]);
    }
    __syncthreads();
    if (kTrain) {
      for (int i = t; i < kIn * 4; i += kNetThreads) {  // X^T, eight rows of a feature each
        const int k = i % kIn, r = 8 * (i / kIn);
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = sx[(r + e) * kXStride + k];
        *reinterpret_cast<uint4*>(out.XT + fragment(k, row0 + r, out.steps)) =
            make_uint4(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16, v[4] | (uint32_t)v[5] << 16,
                       v[6] | (uint32_t)v[7] << 16);
      }
    }
    // layer 1
    f32x16 acc = w1.product(sx + c * kXStride + 8 * half);
    w2.load(W2t + wave * 32 * kHidden + 8 * lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint16_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = activate<kTrain>(acc[4 * q + e] + b1);
        sa[(8 * q + 4 * half + e) * kAStride + n] = v[e];
      }
      if (kTrain)
        *reinterpret_cast<uint2*>(out.A1T + fragment(n, row0 + 8 * q + 4 * half, out.steps)) =
            make_uint2(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16);
    }
    __syncthreads();
    // layer 2
    acc = w2.product(sa + c * kAStride + 8 * half);
    if (kTrain) w2.load(W2b + wave * 32 * kHidden + 8 * lane);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sb[(8 * q + 4 * half + e) * kAStride + n] = activate<kTrain>(acc[4 * q + e] + b2);
    __syncthreads();
    // layer 3: 16 threads a row, 16 hidden units each, then pairwise (a thread a row took 5,200
    // of the forward pass's 16,000 cycles)
    {
      const int r = t / 16, k0 = 16 * (t % 16);
      float z = 0.0f;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint4 w = *reinterpret_cast<const uint4*>(sb + r * kAStride + k0 + 8 * q);
        const uint32_t h[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          z += __uint_as_float(h[e] << 16) * w3[k0 + 8 * q + 2 * e];
          z += __uint_as_float(h[e] & 0xffff0000u) * w3[k0 + 8 * q + 2 * e + 1];
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) z += __shfl_xor(z, o, kWave);
      z += b3;
      const int64_t row = row0 + r;
      if (!kTrain) {
        if (t % 16 == 0 && row < B) logits[row] = z;
      } else if (t % 16 == 0) {
        float dz = 0.0f, l = 0.0f;
        if (row < B) {
          const float yb = y[row];
          dz = (1.0f / (1.0f + expf(-z)) - yb) / (float)B;
          l = (fmaxf(z, 0.0f) - z * yb + log1pf(expf(-fabsf(z)))) / (float)B;
        }
        sdz[r] = dz;
        sloss[r] = l;
      }
    }
    if (!kTrain) return;  // one tile a workgroup
    __syncthreads();
    // dZ2 = bf16(dz w3^T [Z2 > 0]) over X; gw3, gb2 (16 rows a thread), gb3 and the loss
    {
      const int col = t % kHidden, r0 = 16 * (t / kHidden);
      const float w = w3[col];
      uint16_t v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint16_t a2 = sb[(r0 + r) * kAStride + col];
        const float dz = sdz[r0 + r];
        g3 += from_bf16(a2) * dz;
        v[r] = to_bf16(a2 & 0x8000u ? 0.0f : dz * w);
        g2 += from_bf16(v[r]);
        sx[(r0 + r) * kAStride + col] = v[r];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
        *reinterpret_cast<uint4*>(out.dZ2T + fragment(col, row0 + r0 + 8 * q, out.steps)) =
            make_uint4(v[8 * q] | (uint32_t)v[8 * q + 1] << 16, v[8 * q + 2] | (uint32_t)v[8 * q + 3] << 16,
                       v[8 * q + 4] | (uint32_t)v[8 * q + 5] << 16, v[8 * q + 6] | (uint32_t)v[8 * q + 7] << 16);
      if (t < kRows) {  // pairwise over the rows (thread 0's sums count)
        float d = sdz[t], l = sloss[t];
#pragma unroll
        for (int o = kRows / 2; o > 0; o >>= 1) {
          d += __shfl_xor(d, o, kWave);
          l += __shfl_xor(l, o, kWave);
        }
        gb3 += d;
        gl += l;
      }
    }
    __syncthreads();
    // dZ1 = bf16(dZ2 W2^T [Z1 > 0]): element (k, n) of W2^T is W2b[n][k]
    acc = w2.product(sx + c * kAStride + 8 * half);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint16_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = to_bf16(sa[(8 * q + 4 * half + e) * kAStride + n] & 0x8000u ? 0.0f : acc[4 * q + e]);
        g1 += from_bf16(v[e]);
      }
      *reinterpret_cast<uint2*>(out.dZ1T + fragment(n, row0 + 8 * q + 4 * half, out.steps)) =
          make_uint2(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16);
    }
    __syncthreads();  // sx, sa and sb are read: the next tile may write them
  }
  if (kTrain) {
    float* cs = out.colsum + (int64_t)blockIdx.x * kColSums;
    g1 += __shfl_xor(g1, 32, kWave);
    if (half == 0) cs[n] = g1;
    // the two row halves of gb2 and gw3 meet in LDS
    float* meet = reinterpret_cast<float*>(sx);
    if (t >= kHidden) {
      meet[t - kHidden] = g2;
      meet[t] = g3;
    }
    __syncthreads();
    if (t < kHidden) {
      cs[kHidden + t] = g2 + meet[t];
      cs[2 * kHidden + t] = g3 + meet[kHidden + t];
    }
    if (t == 0) {
      cs[3 * kHidden] = gb3;
      cs[3 * kHidden + 1] = gl;
    }
  }
}

// Weight gradients, one split of the batch: rows 0 .. 287 are gW1 = X^T dZ1, rows 288 ..
// 543 gW2 = A1^T dZ2, each element the sum over the split's batch rows.  A workgroup takes 32
// rows x 256 columns, a wave two 32 x 32 blocks; the next eight steps' operands are in flight at once.
__global__ void __launch_bounds__(kThreads, 2) k_wgrad(int64_t steps, int64_t per, TrainOut in,
                                                       float* __restrict__ part) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int c = lane & 31, half = lane >> 5;
  const int m0 = 32 * blockIdx.x;
  const bool first = m0 < kIn;
  const int64_t block = 512 * in.steps;
  const uint16_t* a = (first ? in.XT + m0 / 32 * block : in.A1T + (m0 - kIn) / 32 * block) + 8 * lane;
  const uint16_t* b0 = (first ? in.dZ1T : in.dZ2T) + 2 * wave * block + 8 * lane;
  const uint16_t* b1 = b0 + block;
  const int64_t k0 = (int64_t)blockIdx.y * per, k1 = k0 + per < steps ? k0 + per : steps;
  f32x16 x, y;
#pragma unroll
  for (int r = 0; r < 16; ++r) x[r] = y[r] = 0.0f;
  int64_t k = k0;
  for (; k + 8 <= k1; k += 8) {
    bf16x8 av[8], bv[8], cv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      av[j] = load8(a + 512 * (k + j));
      bv[j] = load8(b0 + 512 * (k + j));
      cv[j] = load8(b1 + 512 * (k + j));
    }
    __builtin_amdgcn_sched_barrier(0);  // all 24 loads in flight
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[j], bv[j], x, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[j], cv[j], y, 0, 0, 0);
    }
  }
  for (; k < k1; ++k) {
    const bf16x8 av = load8(a + 512 * k);
    x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, load8(b0 + 512 * k), x, 0, 0, 0);
    y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, load8(b1 + 512 * k), y, 0, 0, 0);
  }
  float* p = part + (int64_t)blockIdx.y * kGradRows * kHidden;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t row = m0 + 8 * (r >> 2) + 4 * half + (r & 3);
    p[row * kHidden + 64 * wave + c] = x[r];
    p[row * kHidden + 64 * wave + 32 + c] = y[r];
  }
}

// Adam (kTrain of the step) on one parameter.
struct AdamArgs {
  float* m;
  float* v;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ float adam(const AdamArgs& a, int64_t i, float p, float g) {
  const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * g;
  const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * g * g;
  a.m[i] = mi;
  a.v[i] = vi;
  return p - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

// The gradient of every parameter, from the splits (in their order) and the workgroups'
// column sums (lane l of a column's eight adds workgroups l, l + 8, ... in order, then the
// lanes pairwise).  kStep: the Adam step and the bf16 copies of the new weights; else the
// gradients go to G.  Workgroups [0, kGradRows * 256 / kThreads) take the weights, the others
// the column sums.
template <bool kStep>
__global__ void __launch_bounds__(kThreads) k_update(int splits, int groups, const float* __restrict__ part,
                                                    const float* __restrict__ colsum, float* __restrict__ G,
                                                    float* __restrict__ P, AdamArgs ad, uint16_t* __restrict__ W1t,
                                                    uint16_t* __restrict__ W2b, uint16_t* __restrict__ W2t,
                                                    uint16_t* __restrict__ w3b, float* __restrict__ loss) {
  constexpr int kWeightBlocks = kGradRows * kHidden / kThreads;
  if (blockIdx.x < kWeightBlocks) {
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    float s = 0.0f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) s += part[(int64_t)z * kGradRows * kHidden + e];
    const int row = (int)(e / kHidden), n = (int)(e % kHidden);
    const bool first = row < kIn;
    const int k = first ? row : row - kIn;
    const int64_t i = (first ? kOffW1 : kOffW2) + (int64_t)k * kHidden + n;
    if (!kStep) {
      G[i] = s;
      return;
    }
    const float p = adam(ad, i, P[i], s);
    P[i] = p;
    const uint16_t b = to_bf16(p);
    if (first) {
      W1t[fragment(n, k, kIn / 16)] = b;
    } else {
      W2b[fragment(k, n, kHidden / 16)] = b;
      W2t[fragment(n, k, kHidden / 16)] = b;
    }
    return;
  }
  const int t = (blockIdx.x - kWeightBlocks) * kThreads + threadIdx.x;
  const int col = t / 8, l = t % 8;
  float s = 0.0f;
  if (col < kColSums)
#pragma unroll 4
    for (int w = l; w < groups; w += 8) s += colsum[(int64_t)w * kColSums + col];
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
  if (col >= kColSums || l != 0) return;
  if (col == kColSums - 1) {
    *loss = s;
    return;
  }
  const int64_t i = col < kHidden ? kOffB1 + col
                                  : (col < 2 * kHidden ? kOffB2 + (col - kHidden) : kOffW3 + (col - 2 * kHidden));
  if (!kStep) {
    G[i] = s;
    return;
  }
  const float p = adam(ad, i, P[i], s);
  P[i] = p;
  if (col >= 2 * kHidden && col < 3 * kHidden) w3b[col - 2 * kHidden] = to_bf16(p);
}

// bf16 copies of the weights in fragment order: W2b by rows (the backward product dZ2 W2^T),
// W1t / W2t by columns (the forward products).
__global__ void k_refresh(const float* __restrict__ P, uint16_t* __restrict__ W1t, uint16_t* __restrict__ W2b,
                          uint16_t* __restrict__ W2t, uint16_t* __restrict__ w3b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)kIn * kHidden) {
    const int64_t k = i / kHidden, n = i % kHidden;
    W1t[fragment(n, k, kIn / 16)] = to_bf16(P[kOffW1 + i]);
  }
  if (i < (int64_t)kHidden * kHidden) {
    const int64_t k = i / kHidden, n = i % kHidden;
    const uint16_t b = to_bf16(P[kOffW2 + i]);
    W2b[fragment(k, n, kHidden / 16)] = b;
    W2t[fragment(n, k, kHidden / 16)] = b;
  }
  if (i < kHidden) w3b[i] = to_bf16(P[kOffW3 + i]);
}

inline unsigned nblocks(int64_t n, int per = kThreads) { return (unsigned)((n + per - 1) / per > 0 ? (n + per - 1) / per : 1); }

}  // namespace

struct pirrt_mlp {
  int device = 0;
  hipStream_t stream = nullptr;
  int32_t in_dim = 0, max_batch = 0, bcap = 0;
  float lr = 1e-3f, beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
  int64_t t = 0;
  float* P = nullptr;
  float* G = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  uint16_t* W1t = nullptr;  // bf16 W1 by columns, in fragment order
  uint16_t* W2b = nullptr;  // bf16 W2 by rows
  uint16_t* W2t = nullptr;  // bf16 W2 by columns
  uint16_t* w3b = nullptr;
  float* xin = nullptr;   // staging of host features
  float* yin = nullptr;
  float* z = nullptr;     // logits on their way to host memory
  TrainOut T = {};        // operands of the weight gradients, column sums
  float* part = nullptr;  // the weight gradients' splits
  float* hloss = nullptr;  // pinned
  bool poisoned = false;
  std::string err;
};

namespace {

thread_local std::string g_mlp_create_error;

int mfail(pirrt_mlp* N, int code, const std::string& m) {
  N->err = m;
  return code;
}

int mdev(pirrt_mlp* N, hipError_t e, const char* what) {
  N->poisoned = true;
  N->err = std::string("HIP error in ") + what + ": " + hipGetErrorString(e);
  return PIRRT_EDEVICE;
}

#define MHIP(N, expr)                                 \
  do {                                                \
    hipError_t e_ = (expr);                           \
    if (e_ != hipSuccess) return mdev(N, e_, #expr);  \
  } while (0)

template <class T>
bool malloc_dev(T** p, int64_t count) {
  *p = nullptr;
  if (hipMalloc((void**)p, sizeof(T) * (size_t)(count > 0 ? count : 1)) != hipSuccess) {
    (void)hipGetLastError();
    *p = nullptr;
    return false;
  }
  return true;
}

template <class T>
void free_dev(T*& p) {
  if (p) (void)hipFree(p);
  p = nullptr;
}

void release(pirrt_mlp* N) {
  free_dev(N->P); free_dev(N->G); free_dev(N->m); free_dev(N->v); free_dev(N->W1t); free_dev(N->W2b);
  free_dev(N->W2t);
  free_dev(N->w3b); free_dev(N->xin); free_dev(N->yin); free_dev(N->z); free_dev(N->T.XT); free_dev(N->T.A1T);
  free_dev(N->T.dZ1T); free_dev(N->T.dZ2T); free_dev(N->T.colsum);
  free_dev(N->part);
  if (N->hloss) (void)hipHostFree(N->hloss);
  N->hloss = nullptr;
}

int mguard(pirrt_mlp* N) {
  if (!N) return PIRRT_EINVAL;
  if (N->poisoned) return PIRRT_EDEVICE;
  hipError_t e = hipSetDevice(N->device);
  if (e != hipSuccess) return mdev(N, e, "hipSetDevice");
  return PIRRT_OK;
}

// Host features and labels through the handle's staging buffers.
int stage_inputs(pirrt_mlp* N, int32_t B, const float* x, const float* y, int mem_kind, const float** xd,
                 const float** yd) {
  hipStream_t s = N->stream;
  *xd = x;
  *yd = y;
  if (mem_kind == PIRRT_MEM_HOST) {
    MHIP(N, hipMemcpyAsync(N->xin, x, sizeof(float) * (size_t)B * N->in_dim, hipMemcpyHostToDevice, s));
    *xd = N->xin;
    if (y) {
      MHIP(N, hipMemcpyAsync(N->yin, y, sizeof(float) * (size_t)B, hipMemcpyHostToDevice, s));
      *yd = N->yin;
    }
  }
  return PIRRT_OK;
}

inline int32_t row_tiles(int32_t B) { return (B + kRows - 1) / kRows; }

void enqueue_forward(pirrt_mlp* N, int32_t B, const float* xd, float* logits) {
  const int32_t tiles = row_tiles(B);
  hipLaunchKernelGGL(k_net<false>, dim3((unsigned)tiles), dim3(kNetThreads), 0, N->stream, B, tiles, N->in_dim, xd,
                     N->W1t, N->W2t, N->W2b, N->w3b, N->P, nullptr, logits, TrainOut{});
}

// Forward, loss and backward; then the gradients into G, or with `step` one Adam step.  The
// loss lands in N->hloss (pinned: the kernel writes it there).
int enqueue_training(pirrt_mlp* N, int32_t B, const float* xd, const float* yd, float* G, const AdamArgs* step) {
  hipStream_t s = N->stream;
  const int32_t tiles = row_tiles(B), groups = std::min(tiles, (int32_t)kNetGroups);
  hipLaunchKernelGGL(k_net<true>, dim3((unsigned)groups), dim3(kNetThreads), 0, s, B, tiles, N->in_dim, xd, N->W1t,
                     N->W2t, N->W2b, N->w3b, N->P, yd, nullptr, N->T);
  // splits of at least 256 rows; up to 8,192 rows eight of them (136 workgroups, half the partial
  // sums to write: 8.2 us for 4,096 rows, 10.0 with 16), beyond that enough to fill the chip
  const int64_t steps = (int64_t)tiles * (kRows / 16);
  const int64_t want = std::min<int64_t>(steps > 512 ? kSplits : kSplits / 2, (steps + 15) / 16), per = (steps + want - 1) / want;
  const int splits = (int)((steps + per - 1) / per);
  hipLaunchKernelGGL(k_wgrad, dim3(kGradRows / 32, (unsigned)splits), dim3(kThreads), 0, s, steps, per, N->T, N->part);
  const dim3 grid((unsigned)(kGradRows * kHidden / kThreads + (kColSums * 8 + kThreads - 1) / kThreads));
  if (step)
    hipLaunchKernelGGL(k_update<true>, grid, dim3(kThreads), 0, s, splits, groups, N->part, N->T.colsum, nullptr, N->P,
                       *step, N->W1t, N->W2b, N->W2t, N->w3b, N->hloss);
  else
    hipLaunchKernelGGL(k_update<false>, grid, dim3(kThreads), 0, s, splits, groups, N->part, N->T.colsum, G, N->P,
                       AdamArgs{}, N->W1t, N->W2b, N->W2t, N->w3b, N->hloss);
  MHIP(N, hipGetLastError());
  return PIRRT_OK;
}

int check_batch(pirrt_mlp* N, int32_t B, const float* x, int mem_kind) {
  if (mem_kind != PIRRT_MEM_HOST && mem_kind != PIRRT_MEM_DEVICE) return mfail(N, PIRRT_EINVAL, "bad mem_kind");
  if (B < 1 || B > N->max_batch) return mfail(N, PIRRT_EINVAL, "batch size outside 1..max_batch");
  if (!x) return mfail(N, PIRRT_EINVAL, "x is NULL");
  return PIRRT_OK;
}

}  // namespace

extern "C" {

int64_t pirrt_mlp_num_params(void) { return kNumParams; }

int32_t pirrt_mlp_in_dim(const pirrt_mlp* N) { return N ? N->in_dim : -1; }

int pirrt_mlp_create(pirrt_mlp** out, const pirrt_mlp_config* cfg) {
  if (!out || !cfg) return PIRRT_EINVAL;
  *out = nullptr;
  if (cfg->in_dim < 1 || cfg->in_dim > kIn || cfg->max_batch < 1 || cfg->max_batch > (1 << 24) ||
      !(cfg->lr > 0.0f) || !(cfg->beta1 >= 0.0f && cfg->beta1 < 1.0f) || !(cfg->beta2 >= 0.0f && cfg->beta2 < 1.0f) ||
      !(cfg->eps > 0.0f)) {
    g_mlp_create_error = "in_dim outside 1..288, max_batch outside 1..2^24, or bad Adam constants";
    return PIRRT_EINVAL;
  }
  pirrt_mlp* N = new (std::nothrow) pirrt_mlp();
  if (!N) return PIRRT_ENOMEM;
  int dev = cfg->device;
  if ((dev < 0 && hipGetDevice(&dev) != hipSuccess) || hipSetDevice(dev) != hipSuccess) {
    (void)hipGetLastError();
    delete N;
    g_mlp_create_error = "no HIP device";
    return PIRRT_EDEVICE;
  }
  N->device = dev;
  N->stream = (hipStream_t)cfg->hip_stream;
  N->in_dim = cfg->in_dim;
  N->max_batch = cfg->max_batch;
  N->bcap = row_tiles(cfg->max_batch) * kRows;
  N->lr = cfg->lr;
  N->beta1 = cfg->beta1;
  N->beta2 = cfg->beta2;
  N->eps = cfg->eps;
  const int64_t bc = N->bcap;
  bool ok = malloc_dev(&N->P, kNumParams) && malloc_dev(&N->G, kNumParams) && malloc_dev(&N->m, kNumParams) &&
            malloc_dev(&N->v, kNumParams) && malloc_dev(&N->W1t, (int64_t)kIn * kHidden) &&
            malloc_dev(&N->W2b, (int64_t)kHidden * kHidden) && malloc_dev(&N->W2t, (int64_t)kHidden * kHidden) &&
            malloc_dev(&N->w3b, kHidden) &&
            malloc_dev(&N->xin, (int64_t)N->max_batch * N->in_dim) && malloc_dev(&N->yin, N->max_batch) &&
            malloc_dev(&N->z, bc) && malloc_dev(&N->T.XT, bc * kIn) && malloc_dev(&N->T.A1T, bc * kHidden) &&
            malloc_dev(&N->T.dZ1T, bc * kHidden) && malloc_dev(&N->T.dZ2T, bc * kHidden) &&
            malloc_dev(&N->T.colsum, (int64_t)kNetGroups * kColSums) &&
            malloc_dev(&N->part, (int64_t)kSplits * kGradRows * kHidden);
  N->T.steps = bc / 16;
  if (ok && hipHostMalloc((void**)&N->hloss, sizeof(float), hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    N->hloss = nullptr;
    ok = false;
  }
  if (ok)
    ok = hipMemset(N->P, 0, sizeof(float) * kNumParams) == hipSuccess &&
         hipMemset(N->m, 0, sizeof(float) * kNumParams) == hipSuccess &&
         hipMemset(N->v, 0, sizeof(float) * kNumParams) == hipSuccess &&
         hipMemset(N->W1t, 0, sizeof(uint16_t) * kIn * kHidden) == hipSuccess &&
         hipMemset(N->W2b, 0, sizeof(uint16_t) * kHidden * kHidden) == hipSuccess &&
         hipMemset(N->W2t, 0, sizeof(uint16_t) * kHidden * kHidden) == hipSuccess &&
         hipMemset(N->w3b, 0, sizeof(uint16_t) * kHidden) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    release(N);
    delete N;
    g_mlp_create_error = "device allocation failed at create";
    return PIRRT_ENOMEM;
  }
  *out = N;
  return PIRRT_OK;
}

int pirrt_mlp_destroy(pirrt_mlp* N) {
  if (!N) return PIRRT_OK;
  (void)hipSetDevice(N->device);
  if (!N->poisoned) (void)hipStreamSynchronize(N->stream);
  release(N);
  delete N;
  return PIRRT_OK;
}

const char* pirrt_mlp_last_error(const pirrt_mlp* N) { return N ? N->err.c_str() : g_mlp_create_error.c_str(); }

int pirrt_mlp_set_params(pirrt_mlp* N, const float* params, int mem_kind) {
  int rc = mguard(N);
  if (rc) return rc;
  if (mem_kind != PIRRT_MEM_HOST && mem_kind != PIRRT_MEM_DEVICE) return mfail(N, PIRRT_EINVAL, "bad mem_kind");
  if (!params) return mfail(N, PIRRT_EINVAL, "params is NULL");
  if (mem_kind == PIRRT_MEM_HOST)
    for (int64_t i = 0; i < kNumParams; ++i)
      if (!std::isfinite(params[i])) return mfail(N, PIRRT_EINVAL, "parameter not finite");
  hipStream_t s = N->stream;
  MHIP(N, hipMemcpyAsync(N->P, params, sizeof(float) * kNumParams,
                         mem_kind == PIRRT_MEM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice, s));
  MHIP(N, hipMemsetAsync(N->m, 0, sizeof(float) * kNumParams, s));
  MHIP(N, hipMemsetAsync(N->v, 0, sizeof(float) * kNumParams, s));
  hipLaunchKernelGGL(k_refresh, dim3(nblocks((int64_t)kIn * kHidden)), dim3(kThreads), 0, s, N->P, N->W1t, N->W2b,
                     N->W2t, N->w3b);
  MHIP(N, hipGetLastError());
  MHIP(N, hipStreamSynchronize(s));
  N->t = 0;
  return PIRRT_OK;
}

int pirrt_mlp_get_params(pirrt_mlp* N, float* params, int mem_kind) {
  int rc = mguard(N);
  if (rc) return rc;
  if (mem_kind != PIRRT_MEM_HOST && mem_kind != PIRRT_MEM_DEVICE) return mfail(N, PIRRT_EINVAL, "bad mem_kind");
  if (!params) return mfail(N, PIRRT_EINVAL, "params is NULL");
  MHIP(N, hipMemcpyAsync(params, N->P, sizeof(float) * kNumParams,
                         mem_kind == PIRRT_MEM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice, N->stream));
  MHIP(N, hipStreamSynchronize(N->stream));
  return PIRRT_OK;
}

int pirrt_mlp_forward(pirrt_mlp* N, int32_t B, const float* x, float* logits, int mem_kind) {
  int rc = mguard(N);
  if (rc) return rc;
  if ((rc = check_batch(N, B, x, mem_kind))) return rc;
  if (!logits) return mfail(N, PIRRT_EINVAL, "logits is NULL");
  const float *xd = nullptr, *yd = nullptr;
  if ((rc = stage_inputs(N, B, x, nullptr, mem_kind, &xd, &yd))) return rc;
  const bool dev = mem_kind == PIRRT_MEM_DEVICE;
  enqueue_forward(N, B, xd, dev ? logits : N->z);
  MHIP(N, hipGetLastError());
  if (!dev) MHIP(N, hipMemcpyAsync(logits, N->z, sizeof(float) * (size_t)B, hipMemcpyDeviceToHost, N->stream));
  MHIP(N, hipStreamSynchronize(N->stream));
  return PIRRT_OK;
}

int pirrt_mlp_forward_noalloc(pirrt_mlp* N, int32_t B, const float* x, float* logits) {
  int rc = mguard(N);
  if (rc) return rc;
  if (B < 1 || B > PIRRT_MLP_NOALLOC_MAX_BATCH)
    return mfail(N, PIRRT_EINVAL, "batch size outside 1..PIRRT_MLP_NOALLOC_MAX_BATCH");
  if (!x || !logits) return mfail(N, PIRRT_EINVAL, "x or logits is NULL");
  enqueue_forward(N, B, x, logits);
  MHIP(N, hipGetLastError());
  return PIRRT_OK;
}

int pirrt_mlp_gradients(pirrt_mlp* N, int32_t B, const float* x, const float* y, float* grads, float* loss,
                        int mem_kind) {
  int rc = mguard(N);
  if (rc) return rc;
  if ((rc = check_batch(N, B, x, mem_kind))) return rc;
  if (!y) return mfail(N, PIRRT_EINVAL, "y is NULL");
  const float *xd = nullptr, *yd = nullptr;
  if ((rc = stage_inputs(N, B, x, y, mem_kind, &xd, &yd))) return rc;
  const bool dev = mem_kind == PIRRT_MEM_DEVICE;
  if ((rc = enqueue_training(N, B, xd, yd, dev && grads ? grads : N->G, nullptr))) return rc;
  if (grads && !dev)
    MHIP(N, hipMemcpyAsync(grads, N->G, sizeof(float) * kNumParams, hipMemcpyDeviceToHost, N->stream));
  MHIP(N, hipStreamSynchronize(N->stream));
  if (loss) *loss = *N->hloss;
  return PIRRT_OK;
}

int pirrt_mlp_train_step(pirrt_mlp* N, int32_t B, const float* x, const float* y, float* loss, int mem_kind) {
  int rc = mguard(N);
  if (rc) return rc;
  if ((rc = check_batch(N, B, x, mem_kind))) return rc;
  if (!y) return mfail(N, PIRRT_EINVAL, "y is NULL");
  const float *xd = nullptr, *yd = nullptr;
  if ((rc = stage_inputs(N, B, x, y, mem_kind, &xd, &yd))) return rc;
  N->t += 1;
  const AdamArgs step{N->m, N->v, N->lr, N->beta1, N->beta2, N->eps, 1.0f - powf(N->beta1, (float)N->t),
                      1.0f - powf(N->beta2, (float)N->t)};
  if ((rc = enqueue_training(N, B, xd, yd, nullptr, &step))) return rc;
  MHIP(N, hipStreamSynchronize(N->stream));
  if (loss) *loss = *N->hloss;
  return PIRRT_OK;
}

}  // extern "C"
