// Learned collision surrogate: training (forward, backward, Adam) and inference fused into the
// D2Q9 stream-collide step, on bfloat16 matrix cores with float32 accumulation. See
// mlp_common.h for the network, the transposed GEMM formulation and the register layouts.
//
// Training of one batch is two launches: k_mlp_grad (forward and backward, one workgroup per
// 64 samples, per-workgroup partial gradients: the weight gradients are split along the
// sample dimension, K) and k_mlp_reduce_adam (deterministic sum of the partials in a fixed
// order, then the Adam update of the float32 master weights).
#include "mlp_common.h"

#include <algorithm>
#include <cfloat>
#include <cstdlib>
#include <mutex>

#include "lbm.h"

namespace lbm {

constexpr int kPart = kNParam + 1;  // parameters + loss

// Orders this wave's LDS writes before other lanes of the same wave read them: LDS operations
// of one wave execute in order, so only the compiler has to be kept from moving memory
// operations across this point (no workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- forward and backward of one batch -----------------------------------------------------
// LDS of one workgroup: weights (bfloat16, also transposed for the backward products) and biases,
// and the [feature][sample] operands of the weight gradients. Rows of 20 and 68 elements start on
// distinct LDS banks. dL/dZ is kept as its two factors dL/dH and dH/dZ: the biases' gradients sum
// the products with one rounding each (fma), the weight gradients round them to bfloat16. What
// the forward pass alone uses makes room for one of them.
struct __attribute__((aligned(16))) GradForward {
  float b1[kHid], b2[kHid], b3[16];
  short w1[kHid][kW1S], w2[kHid][kW2S], w3[16][kW2S];
  short x[64][kW1S];  // inputs [sample][feature]
};
struct __attribute__((aligned(16))) GradLds {
  union {
    GradForward f;
    float g2[kHid][kW2S];  // dL/dH2^T
  };
  float s2[kHid][kW2S];                    // dH2/dZ2^T
  float g1[kHid][kW2S], s1[kHid][kW2S];  // dL/dH1^T, dH1/dZ1^T
  short w2t[kHid][kW2S], w3t[kHid][kW1S];
  short xt[16][kW2S], dy[16][kW2S];  // X^T, dL/dY^T
  short h1[kHid][kW2S], h2[kHid][kW2S];
  float y[64][20];
  double db3[4][16], loss[4];  // per wavefront
};
static_assert(sizeof(GradLds) <= 160 * 1024, "the LDS of a compute unit");

// Sum over the 16 lanes of a row, in every lane: four rotations within the row, which the vector
// unit reads directly (a shuffle through LDS costs its latency each time).
template <int N>
__device__ __forceinline__ int row_rotate(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false);
}
template <int N>
__device__ __forceinline__ float row_rotate(float v) {
  return __int_as_float(row_rotate<N>(__float_as_int(v)));
}
template <int N>
__device__ __forceinline__ double row_rotate(double v) {
  return __hiloint2double(row_rotate<N>(__double2hiint(v)), row_rotate<N>(__double2loint(v)));
}
template <typename R>
__device__ __forceinline__ R row_sum(R v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  v += row_rotate<1>(v);
  return v;
}

__device__ __forceinline__ float add_rounded(float sum, float a, float b) {
#pragma clang fp contract(off)
  return sum + a * b;
}

// One workgroup of four wavefronts takes the samples (start + i) mod n, i in [64 b, 64 b + 64),
// and writes one row of partial gradients and loss: the weight gradients are split along the
// sample dimension (K). Wavefront v runs the forward and backward passes of samples 16 v ..
// 16 v + 15 (one tile column: a quarter of the matrix and GELU work of 64 samples) and leaves the
// activations and gradients transposed in LDS; after one barrier it forms the weight gradients
// of row tile v over all 64 samples. A batch is bound by latency, not by rate (4096 samples are
// 64 workgroups, and the serial chain of one wavefront is what a step takes): with one wavefront
// for all of its 64 samples and four such wavefronts per compute unit, a training step (this
// kernel and the next) took 44.7 us at 64 samples, 58.5 at 4096 and 289 at 65536; it takes 12.7,
// 13.2 and 51.
__global__ void __launch_bounds__(kBlock)
k_mlp_grad(const float* __restrict__ X, const float* __restrict__ T, int64_t n, int64_t start,
           int B, const float* __restrict__ w, float* __restrict__ partials) {
  __shared__ GradLds s;
  const int t = threadIdx.x;
  const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int first = blockIdx.x * 64;
  // sample k of this workgroup; past the batch: its first one, with zero input and gradient
  auto sample = [&](int k) {
    int64_t i = start + (first + k < B ? first + k : 0);
    if (i >= n) i -= n;
    return i >= n ? i % n : i;
  };

  // weights and inputs into LDS, every load issued before the first write
  {
    float a1[3], a2[16], a3[3], xv[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int e = t + k * kBlock;
      xv[k] = first + e / kIn < B ? X[sample(e / kIn) * kIn + e % kIn] : 0.0f;
      a1[k] = w[oW1 + e];
      a3[k] = e < kOut * kHid ? w[oW3 + e] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) a2[k] = w[oW2 + t + k * kBlock];
    const float b = t < kHid ? w[oB1 + t]
                             : (t < 2 * kHid ? w[oB2 + t - kHid]
                                             : (t < 2 * kHid + kOut ? w[oB3 + t - 2 * kHid] : 0.0f));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int e = t + k * kBlock;
      s.f.w1[e / kIn][e % kIn] = f2bf(a1[k]);
      const short xb = f2bf(xv[k]);
      s.f.x[e / kIn][e % kIn] = xb;
      s.xt[e % kIn][e / kIn] = xb;
      const short wb = f2bf(a3[k]);  // rows 9..11: zero
      s.f.w3[e / kHid][e % kHid] = wb;
      s.w3t[e % kHid][e / kHid] = wb;
    }
    // zero padding: inputs 12..15, outputs 12..15
    s.f.w1[t / 4][kIn + t % 4] = 0;
    s.f.x[t / 4][kIn + t % 4] = 0;
    s.w3t[t / 4][12 + t % 4] = 0;
    s.xt[kIn + t / 64][t % 64] = 0;
    s.f.w3[12 + t / 64][t % 64] = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int e = t + k * kBlock;
      const short v = f2bf(a2[k]);
      s.f.w2[e / kHid][e % kHid] = v;
      s.w2t[e % kHid][e / kHid] = v;
    }
    if (t < kHid) s.f.b1[t] = b;
    else if (t < 2 * kHid) s.f.b2[t - kHid] = b;
    else if (t < 2 * kHid + 16) s.f.b3[t - 2 * kHid] = b;
  }
  __syncthreads();

  const int c = 16 * wv + r;  // this lane's sample
  const bool valid = first + c < B;
  const int64_t idx = sample(c);
  float target[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) target[i] = T[idx * kOut + i];

  // ---- forward ---------------------------------------------------------------------------
  f32x4 z1[4], z2[4];
  bf16x4 h1[4];
  {
    const bf16x4 xb = ld4(&s.f.x[c][4 * q]);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      z1[m] = mfma16(ld4(&s.f.w1[16 * m + r][4 * q]), xb, bias4(s.f.b1 + 16 * m, lane));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h1[m][j] = f2bf(gelu(z1[m][j]));
        s.h1[16 * m + 4 * q + j][c] = h1[m][j];
      }
    }
    bf16x4 h2[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f32x4 acc = bias4(s.f.b2 + 16 * m, lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc = mfma16(ld4(&s.f.w2[16 * m + r][16 * k + 4 * q]), h1[k], acc);
      z2[m] = acc;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h2[m][j] = f2bf(gelu(acc[j]));
        s.h2[16 * m + 4 * q + j][c] = h2[m][j];
      }
    }
    f32x4 y = bias4(s.f.b3, lane);
#pragma unroll
    for (int k = 0; k < 4; ++k) y = mfma16(ld4(&s.f.w3[r][16 * k + 4 * q]), h2[k], y);
#pragma unroll
    for (int j = 0; j < 4; ++j) s.y[c][4 * q + j] = y[j];
  }
  // the outputs of a sample come from its four lanes; g2 takes the place of the forward weights
  __syncthreads();

  // ---- loss and output gradient: every lane of a sample forms all nine, lane q takes 4 q + j --
  bf16x4 dyb;
  {
    float y[9], d[9], dy[9], loss = 0.0f;
#pragma unroll
    for (int i = 0; i < 9; ++i) y[i] = s.y[c][i];
    project9_outputs(y);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      d[i] = valid ? y[i] - target[i] : 0.0f;
      loss += d[i] * d[i];
    }
    // the projection is symmetric: dL/dy = P dL/dyhat
    project9_gradient(d, 2.0f / ((float)B * 9.0f), dy);
    const double l = row_sum((double)loss);
    if (lane == 0) s.loss[wv] = l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float e = q == 0 ? dy[j] : (q == 1 ? dy[4 + j] : (q == 2 && j == 0 ? dy[8] : 0.0f));
      dyb[j] = f2bf(e);
      s.dy[4 * q + j][c] = dyb[j];
      const double v = row_sum((double)e);
      if (r == 0) s.db3[wv][4 * q + j] = v;
    }
  }

  // ---- backward: dH2^T = W3^T dY^T, dZ2 = dH2 gelu'(Z2); dH1^T = W2^T dZ2^T, dZ1 likewise ------
  auto backward = [&](const f32x4& dh, const f32x4& z, float (*gt)[kW2S], float (*st)[kW2S], int m) {
    bf16x4 dz;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float slope = gelu_derivative(z[j]);
      dz[j] = f2bf(dh[j] * slope);
      gt[16 * m + 4 * q + j][c] = dh[j];
      st[16 * m + 4 * q + j][c] = slope;
    }
    return dz;
  };
  bf16x4 dz2[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    dz2[m] = backward(mfma16(ld4(&s.w3t[16 * m + r][4 * q]), dyb, zero), z2[m], s.g2, s.s2, m);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = mfma16(ld4(&s.w2t[16 * m + r][16 * k + 4 * q]), dz2[k], acc);
    backward(acc, z1[m], s.g1, s.s1, m);
  }
  __syncthreads();

  // ---- weight gradients over the 64 samples: row tile wv of W1 and W2, column tile wv of W3 -----
  float* out = partials + (int64_t)blockIdx.x * kPart;
  typedef bf16x4 Rows[4];  // one operand row over the 64 samples
  auto operand = [&](const short* row, Rows& o) {
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = ld4(row + 16 * k + 4 * q);
  };
  auto rounded = [&](const float* g, const float* slope, Rows& o) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(g + 16 * k + 4 * q);
      const f32x4 b = *reinterpret_cast<const f32x4*>(slope + 16 * k + 4 * q);
#pragma unroll
      for (int j = 0; j < 4; ++j) o[k][j] = f2bf(a[j] * b[j]);
    }
  };
  auto product = [&](const Rows& a, const Rows& b) {
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = mfma16(a[k], b[k], acc);
    return acc;
  };
  Rows za, hb;
  rounded(s.g2[16 * wv + r], s.s2[16 * wv + r], za);
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    operand(s.h1[16 * nt + r], hb);
    const f32x4 d = product(za, hb);
#pragma unroll
    for (int j = 0; j < 4; ++j) out[oW2 + (16 * wv + 4 * q + j) * kHid + 16 * nt + r] = d[j];
  }
  rounded(s.g1[16 * wv + r], s.s1[16 * wv + r], za);
  operand(s.xt[r], hb);
  const f32x4 d1 = product(za, hb);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (r < kIn) out[oW1 + (16 * wv + 4 * q + j) * kIn + r] = d1[j];
  operand(s.dy[r], za);
  operand(s.h2[16 * wv + r], hb);
  const f32x4 d3 = product(za, hb);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (4 * q + j < kOut) out[oW3 + (4 * q + j) * kHid + 16 * wv + r] = d3[j];
  // biases: samples 16 apart added in order, then over the 16 lanes of a row. Which products are
  // rounded before they are added (the second layer's, but for units 0, 4, 8 and 12) keeps the
  // results of trainings: either choice is within an ulp of the other, but not after some hundred
  // Adam steps (see gelu_derivative). tests/test_gpu_mlp_pinned.py holds a stored training.
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int h = 16 * wv + 4 * q + j;
    float v1 = 0.0f, v2 = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v1 = __builtin_fmaf(s.g1[h][16 * k + r], s.s1[h][16 * k + r], v1);
      const float g = s.g2[h][16 * k + r], slope = s.s2[h][16 * k + r];
      v2 = wv == 0 && j == 0 ? __builtin_fmaf(g, slope, v2) : add_rounded(v2, g, slope);
    }
    v1 = row_sum(v1);
    v2 = row_sum(v2);
    if (r == 0) {
      out[oB1 + h] = v1;
      out[oB2 + h] = v2;
    }
  }
  if (t < kOut)
    out[oB3 + t] = (float)(((s.db3[0][t] + s.db3[1][t]) + s.db3[2][t]) + s.db3[3][t]);
  else if (t == kBlock - 1)
    out[kNParam] = (float)(((s.loss[0] + s.loss[1]) + s.loss[2]) + s.loss[3]) / ((float)B * 9.0f);
}

// Sum of the partials in row order; optional gradient output and Adam step. A workgroup takes 64
// parameters. Its wavefronts bring kReduceRows rows at a time into LDS, the next ones on their way
// while the first wavefront adds the last ones up: the order of the sum is that of one thread
// reading row after row, which took 16 us for the 64 rows of 4096 samples (22 workgroups, each
// load waited for in small groups).
constexpr int kReduceWaves = 16, kReduceRows = 8 * kReduceWaves;
__global__ void __launch_bounds__(64 * kReduceWaves)
k_mlp_reduce_adam(const float* __restrict__ partials, int nw, float* __restrict__ grad,
                  float* __restrict__ loss, float* __restrict__ w, float* __restrict__ m,
                  float* __restrict__ v, int adam, float lr, float b1, float b2, float eps,
                  float c1, float c2) {
  __shared__ float part[2][kReduceRows][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p = blockIdx.x * 64 + lane;
  const float* col = partials + min(p, kNParam);
  // the parameter and its moments are on their way while the rows are summed
  const bool update = adam && wv == 0 && p < kNParam;
  const float w0 = update ? w[p] : 0.0f, m0 = update ? m[p] : 0.0f, v0 = update ? v[p] : 0.0f;
  float a[8];
  auto fetch = [&](int k0) {  // rows past the last one are read as zero
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = k0 + i * kReduceWaves + wv;
      a[i] = k < nw ? col[(int64_t)k * kPart] : 0.0f;
    }
  };
  fetch(0);
  float g = 0.0f;
  for (int k0 = 0, b = 0; k0 < nw; k0 += kReduceRows, b ^= 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) part[b][i * kReduceWaves + wv][lane] = a[i];
    if (k0 + kReduceRows < nw) fetch(k0 + kReduceRows);
    __syncthreads();
    if (wv == 0) {
      const int n = min(kReduceRows, nw - k0);
      for (int k = 0; k < n; k += 16) {  // rows past nw hold zero
        float r[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) r[i] = part[b][k + i][lane];
#pragma unroll
        for (int i = 0; i < 16; ++i) g += r[i];
      }
    }
  }
  if (wv != 0 || p > kNParam) return;
  if (p == kNParam) {
    if (loss) *loss = g;
    return;
  }
  if (grad) grad[p] = g;
  if (adam) {
    const float mm = __builtin_fmaf(1.0f - b1, g, b1 * m0);
    const float vv = __builtin_fmaf((1.0f - b2) * g, g, b2 * v0);
    m[p] = mm;
    v[p] = vv;
    // bias-corrected moments: c1 = 1 - b1^t, c2 = 1 - b2^t
    w[p] = w0 - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  }
}

// Per-wave LDS rows of the inference kernels: a sample's 12 bfloat16 inputs (zero padded to
// 24) and, once its tile has been evaluated, the same row's 12 float32 outputs (9 used). The
// outputs of tile n overwrite the inputs of tile n only, which that tile has already read.
constexpr int kIoS = 12;  // floats per row (48 bytes)

// Network of one tile (16 samples) of the 64 io rows: inputs in the rows (bfloat16), outputs back
// into the same rows (float32, C layout scattered to rows).
__device__ __forceinline__ void mlp_io_tile(const MlpLdsP& s, float (*io)[kIoS], int nt) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, q = lane >> 4;
  const short(*xs)[2 * kIoS] = reinterpret_cast<const short(*)[2 * kIoS]>(io);
  const f32x4 yt = mlp_forward_tile32<2 * kIoS>(s, xs, nt);
  if (q < 3) {  // output rows 0..11 (9 used)
#pragma unroll
    for (int j = 0; j < 4; ++j) io[16 * nt + r][4 * q + j] = yt[j];
  }
}

// Network of the four tiles of one wave.
__device__ __forceinline__ void mlp_wave_tiles(const MlpLdsP& s, float (*io)[kIoS]) {
#pragma unroll 1
  for (int nt = 0; nt < 4; ++nt) {
    // The weights are re-read from LDS for every tile instead of being hoisted into registers
    // across the tiles (fewer registers, more wavefronts in flight): the byte offset z is 0,
    // but the compiler cannot see it, so the reads stay in the loop. Offsetting the LDS object
    // (rather than laundering the pointer itself) keeps them LDS reads, and every read is the
    // offset base plus an immediate.
    int z = 0;
    asm volatile("" : "+v"(z));
    const MlpLdsP& sz = *reinterpret_cast<const MlpLdsP*>(reinterpret_cast<const char*>(&s) + z);
    mlp_io_tile(sz, io, nt);
  }
}

// A sample's 12 inputs as bfloat16 pairs in the first 6 words of its row, zeros in the next 2
// (the layer-1 tile reads 16 inputs); written as two 16-byte stores (rows are 48-byte aligned).
__device__ __forceinline__ void put_inputs(float* row, const float (&xf)[kIn], bool valid) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  unsigned w[6];
#pragma unroll
  for (int k = 0; k < 6; ++k)
    w[k] = valid ? ((unsigned)(uint16_t)f2bf(xf[2 * k]) | ((unsigned)(uint16_t)f2bf(xf[2 * k + 1]) << 16))
                 : 0u;
  u32x4* r = reinterpret_cast<u32x4*>(__builtin_assume_aligned(row, 16));
  r[0] = u32x4{w[0], w[1], w[2], w[3]};
  r[1] = u32x4{w[4], w[5], 0u, 0u};
}

// Forward pass for n samples (projected outputs), on the inference tiles. SPREAD: one workgroup
// per 64 samples, each wavefront one tile of them, else 64 samples (four tiles) per wavefront.
template <bool SPREAD>
__global__ void __launch_bounds__(kBlock)
k_mlp_forward(const float* __restrict__ X, int64_t n, const float* __restrict__ w, float* __restrict__ Y) {
  __shared__ MlpLdsP s;
  __shared__ __attribute__((aligned(16))) float io[SPREAD ? 1 : 4][64][kIoS];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const bool mine = !SPREAD || wv == 0;  // this wavefront moves inputs and outputs
  const int rows = SPREAD ? 0 : wv;
  const int64_t i = ((int64_t)blockIdx.x * (SPREAD ? 1 : 4) + rows) * 64 + lane;
  const bool valid = i < n;
  if (mine) {
    float xf[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) xf[k] = valid ? X[i * kIn + k] : 0.0f;
    put_inputs(io[rows][lane], xf, valid);
  }
  mlp_load_lds_vec(w, s);
  __syncthreads();  // the weights
  if (SPREAD) {
    mlp_io_tile(s, io[0], wv);
    __syncthreads();
  } else {
    mlp_wave_tiles(s, io[wv]);
    wave_lds_sync();
  }
  if (!mine) return;
  float y[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) y[k] = io[rows][lane][k];
  project9(y);
  if (valid)
#pragma unroll
    for (int k = 0; k < 9; ++k) Y[i * kOut + k] = y[k];
}

// ---- lattice side: harvest and surrogate step ------------------------------------------------
__device__ __forceinline__ double wrest(int i) {
  return (i % 3 == 1 ? 2.0 / 3.0 : 1.0 / 6.0) * (i / 3 == 1 ? 2.0 / 3.0 : 1.0 / 6.0);
}

// Pre-collision shifted values h_i = f_i - w_i at node (x, y) pulled from the state A.
// ROW_UNIFORM: every lane of the wavefront pulls for the same row y (the surrogate step), so
// the source rows are addressed from scalar bases with 32-bit lane offsets; otherwise (the
// harvest, one sampled node per lane) each lane forms its own addresses.
template <bool WALLS, bool ROW_UNIFORM>
__device__ __forceinline__ void pull9h(const float* __restrict__ A, int nx, int ny, int64_t pitch,
                                       int64_t plane, int x, int y, float (&h)[9]) {
  const int xc[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
  const int ys[3] = {y == ny - 1 ? 0 : y + 1, y, y == 0 ? ny - 1 : y - 1};
  if constexpr (ROW_UNIFORM) {
    // byte offsets of the source columns
    const uint32_t xs[3] = {fresh(4u * xc[0]), fresh(4u * xc[1]), fresh(4u * xc[2])};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int ka = i % 3, kb = i / 3;
      const bool bounce = WALLS && ((kb == 2 && y == 0) || (kb == 0 && y == ny - 1));
      const float* row = bounce ? A + (8 - i) * plane + (int64_t)y * pitch
                                : A + i * plane + (int64_t)ys[kb] * pitch;
      h[i] = gload_nt(at_byte(sbase(row), bounce ? xs[1] : xs[ka]));
    }
  } else {
    const int64_t self = (int64_t)y * pitch + x;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int ka = i % 3, kb = i / 3;
      const bool bounce = WALLS && ((kb == 2 && y == 0) || (kb == 0 && y == ny - 1));
      h[i] = bounce ? A[(8 - i) * plane + self] : A[i * plane + (int64_t)ys[kb] * pitch + xc[ka]];
    }
  }
}

// Pre-collision populations at node (x, y) pulled from the shifted float32 state A.
template <bool WALLS>
__device__ __forceinline__ void pull9(const float* __restrict__ A, int nx, int ny, int64_t pitch,
                                      int64_t plane, int x, int y, double (&f)[9]) {
  float h[9];
  pull9h<WALLS, false>(A, nx, ny, pitch, plane, x, y, h);
#pragma unroll
  for (int i = 0; i < 9; ++i) f[i] = (double)h[i] + wrest(i);
}

// Pre-collision populations of the next step at node (x, y) from a stored state of either
// layout: view -1 two-buffer (pull of slot i from x - c_i), 0 single-buffer after an even step
// count (slot 8-i of x - c_i; slot i of x where x - c_i lies beyond a wall), 1 single-buffer
// after an odd step count (slot i of x, already streamed).
template <bool WALLS>
__device__ __forceinline__ void next_input9(const float* __restrict__ A, int nx, int ny,
                                            int64_t pitch, int64_t plane, int view, int x, int y,
                                            double (&f)[9]) {
  if (view < 0) {
    pull9<WALLS>(A, nx, ny, pitch, plane, x, y, f);
    return;
  }
  const int xs[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
  const int ys[3] = {y == ny - 1 ? 0 : y + 1, y, y == 0 ? ny - 1 : y - 1};
  const int64_t self = (int64_t)y * pitch + x;
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int ka = i % 3, kb = i / 3;
    const bool wall = WALLS && ((kb == 2 && y == 0) || (kb == 0 && y == ny - 1));
    float h;
    if (view == 1 || wall)
      h = A[i * plane + self];
    else
      h = A[(8 - i) * plane + (int64_t)ys[kb] * pitch + xs[ka]];
    f[i] = (double)h + wrest(i);
  }
}

template <bool WALLS>
__global__ void k_harvest(const float* __restrict__ A, int nx, int ny, int64_t pitch, int64_t plane,
                          int view, double omega, const int64_t* __restrict__ nodes, int64_t n,
                          float* __restrict__ X, float* __restrict__ Y) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int64_t node = nodes[k];
  const int x = (int)(node % nx), y = (int)(node / nx);
  double f[9];
  next_input9<WALLS>(A, nx, ny, pitch, plane, view, x, y, f);
  const double rho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
  const double ux = ((f[2] + f[5] + f[8]) - (f[0] + f[3] + f[6])) / rho;
  const double uy = ((f[6] + f[7] + f[8]) - (f[0] + f[1] + f[2])) / rho;
  float xf[12];
  mlp_features(f, rho, ux, uy, omega, xf);
#pragma unroll
  for (int i = 0; i < 12; ++i) X[k * kIn + i] = xf[i];
  // plain-collision target S (f~ - f^eq)/rho = (1 - omega) S (f - f^eq)/rho
#pragma unroll
  for (int i = 0; i < 9; ++i) Y[k * kOut + i] = (float)((1.0 - omega) * (double)xf[i]);
}

// One D2Q9 step with the surrogate collision and the per-node plain-collision judge, in float32
// on the shifted values h = f - w (w the rest weights). With theta = 1/3 the per-axis factors
// are psi_c = W_c + d_c, W = (1/6, 2/3, 1/6), d_0 = -u^2, d_+- = (u^2 +- u)/2, and
//   h^eq_i = f^eq_i - w_i = (rho - 1) psi_a psi_b + W_a d_b + d_a W_b + d_a d_b,
// with float32 constants whose sum is exactly one (W_+- = 2796203 2^-24, W_0 = 1 - 2 W_+-:
// with the nearest float32 values of 1/6 and 2/3 the sum of the factors misses one by 3e-8 and
// every collision rescales mass and momentum by that amount).
//   features  x = [1024 (h_i - h^eq_i)/rho, 16 u_x, 16 u_y, omega]
//   network   y (projected), surrogate f~ = f^eq + rho y / 1024
//   judge     |f~_mlp - f~_plain| <= tol |f~_plain - f^eq| with f~_plain - f^eq = (1 - omega)(f - f^eq),
//             i.e. |y - (1 - omega) x_neq| <= tol |1 - omega| |x_neq| (the factor rho / 1024 cancels)
//   fallback  h~ = h + omega (h^eq - h)
// One wavefront evaluates the network for its 64 nodes of a row; only the weights are shared by
// the workgroup (one barrier after their load), the rest of a row is synchronised per wave.
template <bool WALLS, bool DIAG>
__global__ void __launch_bounds__(kBlock)
k_bgk_d2q9_mlp(const float* __restrict__ A, float* __restrict__ B, int nx, int ny, int64_t pitch,
               int64_t plane, float omega, int rows, const float* __restrict__ wblob, float tol2,
               unsigned long long* __restrict__ counters, double* __restrict__ partials) {
  __shared__ MlpLdsP s;
  __shared__ __attribute__((aligned(16))) float io[4][64][kIoS];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nbx = gridDim.x;
  const int tile = xcd_tile(blockIdx.x + nbx * blockIdx.y, nbx * gridDim.y);
  const int bx = tile % nbx, by = tile / nbx;
  const int x = bx * blockDim.x + threadIdx.x;
  const bool valid = x < nx;
  const int y0 = by * rows, yend = min(y0 + rows, ny);
  const float W1 = 2796203.0f / 16777216.0f, W0 = 1.0f - 2.0f * W1;  // exact in float32
  const float keep = 1.0f - omega;
  double acc[kDiagValues] = {0.0, 0.0, 0.0, 0.0, 0.0};
  unsigned fallbacks = 0;
  mlp_load_lds_vec(wblob, s);
  // One row: features, network, judge and store from the pulled populations h of row y.
  // Lanes past the right edge work on the last column's values (pulled from a valid column,
  // so finite) and store nothing: no separate zero-filled path.
  auto row = [&](const float (&h)[9], int y) {
    float heq[9], xf[kIn];
    float drho, ux, uy;
    {
      drho = ((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7])) + h[8];
      const float jx = (h[2] + h[5] + h[8]) - (h[0] + h[3] + h[6]);
      const float jy = (h[6] + h[7] + h[8]) - (h[0] + h[1] + h[2]);
      const float inv = __builtin_amdgcn_rcpf(1.0f + drho);
      // u = j / rho with one residual correction of the hardware reciprocal (unbiased: a
      // one-sided velocity error would shift every node's momentum the same way each step)
      ux = jx * inv;
      uy = jy * inv;
      ux = __builtin_fmaf(__builtin_fmaf(-(1.0f + drho), ux, jx), inv, ux);
      uy = __builtin_fmaf(__builtin_fmaf(-(1.0f + drho), uy, jy), inv, uy);
      const float u2x = ux * ux, u2y = uy * uy;
      const float dx[3] = {0.5f * (u2x - ux), -u2x, 0.5f * (u2x + ux)};
      const float dy[3] = {0.5f * (u2y - uy), -u2y, 0.5f * (u2y + uy)};
      const float Wk[3] = {W1, W0, W1};
      const float sx = kSNeq * inv;
      // the same sum regrouped: h^eq_i = psi_b (drho psi_a + d_a) + W_a d_b (psi = W + d)
      float A[3], P[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        A[k] = __builtin_fmaf(drho, Wk[k] + dx[k], dx[k]);
        P[k] = Wk[k] + dy[k];
      }
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        const int ia = i % 3, ib = i / 3;
        heq[i] = __builtin_fmaf(P[ib], A[ia], Wk[ia] * dy[ib]);
        xf[i] = (h[i] - heq[i]) * sx;
      }
      xf[9] = kSU * ux;
      xf[10] = kSU * uy;
      xf[11] = omega;
    }
    wave_lds_sync();  // the previous row's outputs have been read
    put_inputs(io[wv][lane], xf, true);
    wave_lds_sync();
    mlp_wave_tiles(s, io[wv]);
    wave_lds_sync();
    if (valid) {
      float yv[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) yv[i] = io[wv][lane][i];
      project9(yv);
      float err = 0.0f, ref = 0.0f;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        const float d = yv[i] - keep * xf[i];
        err += d * d;
        ref += xf[i] * xf[i];
      }
      const bool fb = !(err <= tol2 * (keep * keep) * ref);
      fallbacks += fb ? 1u : 0u;
      const float rs = (1.0f + drho) * (1.0f / kSNeq);
      const uint32_t xo = fresh(4u * x);
#pragma unroll
      for (int i = 0; i < 9; ++i)
        gstore_nt(at_byte(sbase(B + i * plane + (int64_t)y * pitch), xo),
                  fb ? h[i] + omega * (heq[i] - h[i]) : heq[i] + rs * yv[i]);
      if (DIAG) {
        const double rho = 1.0 + (double)drho;
        acc[0] += rho;
        acc[1] += rho * (double)ux;
        acc[2] += rho * (double)uy;
        acc[4] += 0.5 * rho * ((double)ux * ux + (double)uy * uy);
      }
    }
  };
  // Rows in pairs with two pull buffers: the populations of the next row are loaded while the
  // network of the current one runs (software pipelining without register copies).
  // The loads are unconditional (lanes past the edge read the last column, a pull past the
  // last row re-reads it), so that the compiler's wait for one buffer never includes the other.
  float ha[9], hb[9];
  const int xl = valid ? x : nx - 1;
  const int ylast = yend - 1;
  if (y0 < yend) pull9h<WALLS, true>(A, nx, ny, pitch, plane, xl, y0, ha);
  __syncthreads();
  for (int y = y0; y < yend; y += 2) {
    pull9h<WALLS, true>(A, nx, ny, pitch, plane, xl, min(y + 1, ylast), hb);
    row(ha, y);
    if (y + 1 >= yend) break;
    pull9h<WALLS, true>(A, nx, ny, pitch, plane, xl, min(y + 2, ylast), ha);
    row(hb, y + 1);
  }
  // integer fallback counts: order-independent, so atomics stay deterministic
  unsigned long long fb = (unsigned long long)fallbacks;
  unsigned long long upd = (unsigned long long)(valid ? yend - y0 : 0);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    fb += __shfl_xor(fb, off, 64);
    upd += __shfl_xor(upd, off, 64);
  }
  if (lane == 0) {
    atomicAdd(counters, fb);
    atomicAdd(counters + 1, upd);
  }
  if (DIAG) block_sum_store<kDiagValues>(acc, partials + (int64_t)tile * kDiagValues);
}

// ---- launchers ---------------------------------------------------------------------------------
hipError_t launch_mlp_grad(const float* X, const float* T, int64_t n, int64_t start, int B,
                           const float* w, float* partials, hipStream_t s) {
  const int nw = (B + 63) / 64;
  k_mlp_grad<<<nw, kBlock, 0, s>>>(X, T, n, start, B, w, partials);
  return hipGetLastError();
}

int mlp_partial_count(int B) { return (B + 63) / 64; }

hipError_t launch_mlp_reduce_adam(const float* partials, int nw, float* grad, float* loss, float* w,
                                  float* m, float* v, bool adam, float lr, int64_t t, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = (float)(1.0 - std::pow(0.9, (double)t));
  const float c2 = (float)(1.0 - std::pow(0.999, (double)t));
  k_mlp_reduce_adam<<<(kNParam + 64) / 64, 64 * kReduceWaves, 0, s>>>(
      partials, nw, grad, loss, w, m, v, adam ? 1 : 0, lr, b1, b2, eps, c1, c2);
  return hipGetLastError();
}

// Workgroups of 64 samples up to 2^18 samples, 64 samples per wavefront above (us, one tile / four
// tiles per wavefront: 64 samples 4.0 / 6.8, 4096 4.3 / 7.2, 65536 6.7 / 7.8, 2^18 19.5 / 20.7,
// 2^20 65.8 / 61.9, 2^22 259 / 218): few workgroups are bound by one wavefront's chain of four
// tiles, many by the loads of the weights, which a workgroup of 256 samples shares.
constexpr int64_t kSpreadForward = 4096;
hipError_t launch_mlp_forward(const float* X, int64_t n, const float* w, float* Y, hipStream_t s) {
  const int64_t nw = (n + 63) / 64;
  if (nw <= kSpreadForward)
    k_mlp_forward<true><<<(unsigned)nw, kBlock, 0, s>>>(X, n, w, Y);
  else
    k_mlp_forward<false><<<(unsigned)((nw + 3) / 4), kBlock, 0, s>>>(X, n, w, Y);
  return hipGetLastError();
}

hipError_t launch_harvest(const void* A, const Layout& L, bool walls, int view, double omega,
                          const int64_t* nodes, int64_t n, float* X, float* Y, hipStream_t s) {
  const unsigned nb = (unsigned)((n + kBlock - 1) / kBlock);
  if (walls)
    k_harvest<true><<<nb, kBlock, 0, s>>>(static_cast<const float*>(A), L.nx, L.ny, L.pitch, L.plane, view, omega, nodes, n, X, Y);
  else
    k_harvest<false><<<nb, kBlock, 0, s>>>(static_cast<const float*>(A), L.nx, L.ny, L.pitch, L.plane, view, omega, nodes, n, X, Y);
  return hipGetLastError();
}

// Workgroups of the surrogate step that the current device holds at once (compute units times
// the workgroups one compute unit holds with this kernel's registers and LDS), or 0 if the
// device cannot be queried.
static int mlp_resident_workgroups() {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_bgk_d2q9_mlp<false, false>, kBlock, 0) !=
      hipSuccess)
    return 0;
  return cus * per;
}

// Rows per workgroup: as few as keep every workgroup resident at once (one round over the
// chip, so no tail of late workgroups), which also spreads the per-workgroup weight load over
// as many rows as possible. 2048^2 on MI355X: 13 rows, 1264 workgroups for 256 x 5 resident.
Grid make_grid_mlp(const Layout& L) {
  Grid G;
  G.bx = kBlock;
  G.nbx = (L.nx + kBlock - 1) / kBlock;
  G.rows = 8;
  const int64_t resident = mlp_resident_workgroups();
  if (resident > 0) {
    const int64_t units = (int64_t)L.ny * G.nbx;
    G.rows = (int)std::max<int64_t>(1, (units + resident - 1) / resident);
  }
#ifdef LBM_TUNING_ENV
  if (const char* v = getenv("LBM_MLP_ROWS")) G.rows = atoi(v);
#endif
  fit_rows(G, L.ny);
  return G;
}

hipError_t launch_bgk_d2q9_mlp(const void* A, void* B, const Layout& L, const Grid& G, double omega_d,
                               bool walls, const float* wblob, double tol_d,
                               unsigned long long* counters, double* partials, hipStream_t s) {
  dim3 grid(G.nbx, G.nby), block(kBlock);
  auto a = static_cast<const float*>(A);
  auto b = static_cast<float*>(B);
  const float omega = (float)omega_d;
  // tol^2 as a finite float32 (a huge tolerance then still gives 0 * tol^2 = 0 where the
  // non-equilibrium part vanishes, as the float64 comparison does)
  const float tol2 = (float)std::min(tol_d * tol_d, (double)FLT_MAX);
  if (walls) {
    if (partials) k_bgk_d2q9_mlp<true, true><<<grid, block, 0, s>>>(a, b, L.nx, L.ny, L.pitch, L.plane, omega, G.rows, wblob, tol2, counters, partials);
    else k_bgk_d2q9_mlp<true, false><<<grid, block, 0, s>>>(a, b, L.nx, L.ny, L.pitch, L.plane, omega, G.rows, wblob, tol2, counters, nullptr);
  } else {
    if (partials) k_bgk_d2q9_mlp<false, true><<<grid, block, 0, s>>>(a, b, L.nx, L.ny, L.pitch, L.plane, omega, G.rows, wblob, tol2, counters, partials);
    else k_bgk_d2q9_mlp<false, false><<<grid, block, 0, s>>>(a, b, L.nx, L.ny, L.pitch, L.plane, omega, G.rows, wblob, tol2, counters, nullptr);
  }
  return hipGetLastError();
}

// ---- gradient without allocation ---------------------------------------------------------------
// For callers that cannot call hipMalloc (graph capture, serving loops): the partial
// gradients of k_mlp_grad go to a fixed device array instead of a trainer buffer. Each
// GPU the library runs on holds its own copy of the array until the process ends; its device
// address is looked up once per device (with that device current) and kept. k_mlp_grad writes
// every entry of the rows it uses, so nothing has to be cleared between calls; calls that
// overlap on one GPU race on the array.
namespace {
constexpr int kStaticMaxSamples = LBM_MLP_STATIC_MAX_SAMPLES;
constexpr int kStaticRows = (kStaticMaxSamples + 63) / 64;
static __device__ __align__(256) float scratch[(size_t)kStaticRows * kPart];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call per device).
hipError_t scratch_on_current_device(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

}  // namespace lbm

extern "C" int lbm_mlp_grad_static(const float* dev_weights, const float* dev_x,
                                   const float* dev_t, int64_t n, float* dev_grad,
                                   float* dev_loss, void* stream) {
  using namespace lbm;
  if (n <= 0 || n > kStaticMaxSamples) return LBM_EINVAL;
  if (!dev_weights || !dev_x || !dev_t || !dev_grad) return LBM_EINVAL;
  static_assert((size_t)kStaticRows * kPart * sizeof(float) <= ((size_t)8 << 20),
                "the fixed partials array stays below 8 MiB");
  float* part = nullptr;
  if (scratch_on_current_device(&part) != hipSuccess) return LBM_EDEVICE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int B = (int)n;
  hipError_t e = launch_mlp_grad(dev_x, dev_t, n, 0, B, dev_weights, part, s);
  // adam = false: the kernel reads the partials and writes grad (and loss); w, m, v untouched
  if (e == hipSuccess)
    e = launch_mlp_reduce_adam(part, mlp_partial_count(B), dev_grad, dev_loss,
                               const_cast<float*>(dev_weights), nullptr, nullptr, false, 0.0f, 1, s);
  return e == hipSuccess ? LBM_OK : LBM_EDEVICE;
}
