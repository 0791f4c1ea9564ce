// proposal.hip - the learned direction proposal's network on the matrix cores: inference
// (features -> 320 -> 64 -> 64 -> 256 -> softmax), one training step (forward, cross
// entropy, backward, weight gradients) and Adam. An extension of the Monte Carlo estimate of
// Eq. 7 (ComGS Sec. 3.1.2): the network's bin distribution is what the proposal sampler of
// shade.hip draws from.
//
// Matrix products run on v_mfma_f32_16x16x32_bf16 in a transposed formulation, z^T = W^T x^T:
// the output neurons are the M dimension and 16 points are the N dimension, so the
// accumulators of one layer (lane l holds rows 4(l/16)..+3 of column l%16), after bias,
// ReLU and rounding, are the B operands of the next layer (two 16-row blocks per 32-input
// block, in the K order of mlp_device.hpp); no shuffles or LDS round trips between layers.
// Weights are pre-arranged once per call into operand fragments (64 lanes x 8 bf16 = 1 KB,
// one coalesced load).
// Weight gradients contract over points, so they use activations stored transposed
// ([feature][point]) and are a plain GEMM in which each workgroup owns one 16x16 tile of a
// weight matrix (deterministic, no atomics).
#include "mlp_device.hpp"

namespace sopk {

// ------------------------------------------------------------------------------------------
// fragment preparation: one thread per bf16 element
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_mlp_frags(const float* __restrict__ P,
                                                   uint16_t* __restrict__ frags) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= kFrags * kFragElems) return;
  const int f = e / kFragElems, lane = (e >> 3) & 63, j = e & 7;
  const int g = lane >> 4, r = lane & 15;
  int src;
  if (f < kF2) {                 // W1^T[out][in]: A[m = out 16mb + r][k = in]
    const int mb = (f - kF1) / 10, kb = (f - kF1) % 10;
    src = kOffW1 + kpos_input(kb, g, j) * kHid + 16 * mb + r;
  } else if (f < kF3) {
    const int mb = (f - kF2) / 2, kb = (f - kF2) % 2;
    src = kOffW2 + kpos_input(kb, g, j) * kHid + 16 * mb + r;
  } else if (f < kB3) {
    const int mb = (f - kF3) / 2, kb = (f - kF3) % 2;
    src = kOffW3 + kpos_input(kb, g, j) * kBins + 16 * mb + r;
  } else if (f < kB2) {          // W3[in][out]: A[m = in 16mb + r][k = out]
    const int mb = (f - kB3) / 8, kb = (f - kB3) % 8;
    src = kOffW3 + (16 * mb + r) * kBins + kpos_input(kb, g, j);
  } else {
    const int mb = (f - kB2) / 2, kb = (f - kB2) % 2;
    src = kOffW2 + (16 * mb + r) * kHid + kpos_input(kb, g, j);
  }
  frags[e] = f2bf(P[src]);
}

// ------------------------------------------------------------------------------------------
// inference: one wavefront per 16 points
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_infer(MlpArgs a) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t p0 = tile * 16;
  if (p0 >= a.n) return;
  const int64_t p = p0 + r;
  const bool valid = p < a.n;
  FeatIn fi;
  if (valid) point_scalars(a.pos, a.nrm, a.view, a.cam, a.ppf, a.rough, a.lo, a.inv2, p, fi);
  else
#pragma unroll
    for (int c = 0; c < 10; ++c) fi.x[c] = 0.0f;
  Fwd F;
  forward_tile(a.params, a.frags, fi, lane, F);
  if (valid && a.logits) {
#pragma unroll
    for (int mb = 0; mb < 16; ++mb)
      *reinterpret_cast<float4*>(a.logits + (size_t)p * kBins + 16 * mb + 4 * g) =
          make_float4(F.z3[mb][0], F.z3[mb][1], F.z3[mb][2], F.z3[mb][3]);
  }
  softmax_tile(F.z3);
  if (!valid) return;
#pragma unroll
  for (int mb = 0; mb < 16; ++mb)
    *reinterpret_cast<float4*>(a.probs + (size_t)p * kBins + 16 * mb + 4 * g) =
        make_float4(F.z3[mb][0], F.z3[mb][1], F.z3[mb][2], F.z3[mb][3]);
}

// ------------------------------------------------------------------------------------------
// training: forward + cross entropy + backward of one 16-point tile per workgroup.
// Writes the transposed bf16 operands of the weight-gradient GEMM (zero for padding points)
// and the tile's bias-gradient column sums and loss, which the weight-gradient kernel adds
// up in a fixed order (no atomics: a step is deterministic).
// A batch of 4096 points is 256 tiles, one per compute unit, and a tile is one chain through
// six layers: what bounds it is the chain, not the arithmetic. Its four wavefronts share every
// layer (wavefront w has the 16 neurons of block w of the hidden layers and 64 of the bins) and
// hand the next layer's operands over in LDS: 15 us, 36 with one wavefront per tile. Batches
// that fill the chip gain as well, by the shorter chain (whole steps, one / four wavefronts per
// tile: 16,384 points 71 / 54 us, 65,536 249 / 178, 262,144 1036 / 821, 1M 5730 / 4999).
// ------------------------------------------------------------------------------------------
constexpr int kPart = kMlpPart;
constexpr int kTrainWaves = 4;

// sum over the 16 points: by row operations
__device__ __forceinline__ float tile_col_sum(float v) {
  v = dpp_add<0xB1>(v);          // quad_perm [1,0,3,2]
  v = dpp_add<0x4E>(v);          // quad_perm [2,3,0,1]
  v = dpp_add<0x141>(v);         // row_half_mirror
  return dpp_add<0x140>(v);      // row_mirror
}

// stores a block's fragment as rows 16 mb + 4 g + t of a transposed operand
__device__ __forceinline__ void store_rows(uint16_t* T, int64_t ldT, int64_t col, int row0,
                                           bf16x4 v) {
#pragma unroll
  for (int t = 0; t < 4; ++t) T[(size_t)(row0 + t) * ldT + col] = (uint16_t)v[t];
}

__global__ __launch_bounds__(64 * kTrainWaves) void k_mlp_train(MlpArgs a) {
  __shared__ bf16x8s s_x[10][64];                // B operands of the first layer
  __shared__ bf16x4 s_h1[4][64], s_h2[4][64], s_d3[16][64], s_d2[4][64];
  __shared__ float s_max[kTrainWaves][16], s_sum[kTrainWaves][16], s_tgt[kTrainWaves][16];
  __shared__ float s_loss[kTrainWaves];
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t tile = blockIdx.x;
  const int64_t p0 = tile * 16;
  if (p0 >= a.ldT) return;                        // ldT = batch rounded up to 32
  const int64_t p = p0 + r;
  const bool valid = p < a.n;
  const float vmask = valid ? 1.0f : 0.0f;
  const int row0 = 16 * w + 4 * g;                // the lane's rows of the wavefront's block
  float* part = a.part + tile * kPart;
  auto operand = [&](const bf16x4 (*v)[64], int kb) {
    return cat8(v[2 * kb][lane], v[2 * kb + 1][lane]);
  };
  // features: scalar kb of the ten
  FeatIn fi;
  if (valid) point_scalars(a.pos, a.nrm, a.view, a.cam, a.ppf, a.rough, a.lo, a.inv2, p, fi);
  else
#pragma unroll
    for (int c = 0; c < 10; ++c) fi.x[c] = 0.0f;
#pragma unroll
  for (int kb = 0; kb < 10; ++kb) {               // fully unrolled: fi.x[kb] stays in registers
    if (kb % kTrainWaves != w) continue;
    const bf16x4 b0 = feature_frag(fi, 2 * kb, g), b1 = feature_frag(fi, 2 * kb + 1, g);
    store_rows(a.xT, a.ldT, p, 32 * kb + 4 * g, b0);
    store_rows(a.xT, a.ldT, p, 32 * kb + 16 + 4 * g, b1);
    s_x[kb][lane] = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  __syncthreads();
  auto bias = [&](int off) {
    f32x4 z;
#pragma unroll
    for (int t = 0; t < 4; ++t) z[t] = a.params[off + t];
    return z;
  };
  auto relu4 = [](const f32x4& z) {
    return pack4(fmaxf(z[0], 0.0f), fmaxf(z[1], 0.0f), fmaxf(z[2], 0.0f), fmaxf(z[3], 0.0f));
  };
  const bf16x4 none = {0, 0, 0, 0};
  f32x4 z1 = bias(kOffB1 + row0);
#pragma unroll
  for (int kb = 0; kb < 10; ++kb)
    z1 = mfma32(load_frag(a.frags, kF1 + w * 10 + kb, lane),
                __builtin_bit_cast(bf16x8, s_x[kb][lane]), z1);
  const bf16x4 h1 = relu4(z1);
  s_h1[w][lane] = h1;
  // activations stored transposed (zero for padding points)
  store_rows(a.h1T, a.ldT, p, row0, valid ? h1 : none);
  __syncthreads();
  f32x4 z2 = bias(kOffB2 + row0);
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
    z2 = mfma32(load_frag(a.frags, kF2 + w * 2 + kb, lane), operand(s_h1, kb), z2);
  const bf16x4 h2 = relu4(z2);
  s_h2[w][lane] = h2;
  store_rows(a.h2T, a.ldT, p, row0, valid ? h2 : none);
  // the targets are loaded meanwhile
  float4 T[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    T[i] = valid ? *reinterpret_cast<const float4*>(a.targets + (size_t)p * kBins +
                                                    16 * (4 * w + i) + 4 * g)
                 : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  __syncthreads();
  f32x4 z3[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) z3[i] = bias(kOffB3 + 16 * (4 * w + i) + 4 * g);
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const bf16x8 b = operand(s_h2, kb);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      z3[i] = mfma32(load_frag(a.frags, kF3 + (4 * w + i) * 2 + kb, lane), b, z3[i]);
  }
  // softmax, normalised targets, loss, dz3 = (q - t) / B
  float mx = -INFINITY, ts = 0.0f, se = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int t = 0; t < 4; ++t) mx = fmaxf(mx, z3[i][t]);
    ts += T[i].x + T[i].y + T[i].z + T[i].w;
  }
  mx = point_max(mx);
  ts = point_sum(ts);
  if (g == 0) {
    s_max[w][r] = mx;
    s_tgt[w][r] = ts;
  }
  __syncthreads();
  mx = fmaxf(fmaxf(s_max[0][r], s_max[1][r]), fmaxf(s_max[2][r], s_max[3][r]));
  ts = (s_tgt[0][r] + s_tgt[1][r]) + (s_tgt[2][r] + s_tgt[3][r]);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int t = 0; t < 4; ++t) se += expf(z3[i][t] - mx);
  se = point_sum(se);
  if (g == 0) s_sum[w][r] = se;
  __syncthreads();
  se = (s_sum[0][r] + s_sum[1][r]) + (s_sum[2][r] + s_sum[3][r]);
  const float lse = mx + logf(se);
  const bool uni = !(ts > 0.0f);
  const float its = uni ? 0.0f : 1.0f / ts;
  const float invB = 1.0f / (float)a.n;
  float loss = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int mb = 4 * w + i;
    const float tv[4] = {T[i].x, T[i].y, T[i].z, T[i].w};
    float dz[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float tt = uni ? (1.0f / kBins) : tv[t] * its;
      loss -= tt * (z3[i][t] - lse);
      dz[t] = (expf(z3[i][t] - lse) - tt) * invB * vmask;
      const float cs = tile_col_sum(dz[t]);
      if (r == 0) part[2 * kHid + 16 * mb + 4 * g + t] = cs;
    }
    const bf16x4 d3 = pack4(dz[0], dz[1], dz[2], dz[3]);
    s_d3[mb][lane] = d3;
    store_rows(a.dz3T, a.ldT, p, 16 * mb + 4 * g, d3);
  }
  loss = wave_sum(loss * vmask);
  if (lane == 0) s_loss[w] = loss;
  __syncthreads();
  if (threadIdx.x == 0)
    part[kPart - 1] = ((s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3])) * invB;
  // dh2^T = W3 dz3^T, dz2 = dh2 [z2 > 0]; then dh1^T = W2 dz2^T, dz1 = dh1 [z1 > 0]
  auto masked = [&](const f32x4& acc, const f32x4& z, int part0) {
    float dz[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      dz[t] = z[t] > 0.0f ? acc[t] : 0.0f;
      const float cs = tile_col_sum(dz[t]);
      if (r == 0) part[part0 + row0 + t] = cs;
    }
    return pack4(dz[0], dz[1], dz[2], dz[3]);
  };
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int kb = 0; kb < 8; ++kb)
    acc = mfma32(load_frag(a.frags, kB3 + w * 8 + kb, lane), operand(s_d3, kb), acc);
  const bf16x4 d2 = masked(acc, z2, kHid);
  s_d2[w][lane] = d2;
  store_rows(a.dz2T, a.ldT, p, row0, d2);
  __syncthreads();
  acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
    acc = mfma32(load_frag(a.frags, kB2 + w * 2 + kb, lane), operand(s_d2, kb), acc);
  store_rows(a.dz1T, a.ldT, p, row0, masked(acc, z1, 0));
}

// ------------------------------------------------------------------------------------------
// weight gradients: dW[in][out] = sum_points act[in][pt] dz[out][pt], one 16x16 tile per
// workgroup, K = the (padded) batch. There are only 160 tiles and a tile is one serial chain
// of loads over the batch, so kWgWaves wavefronts share it: each sums its part of the points,
// the parts are added in LDS in a fixed order (so that a training step is deterministic).
// Batch of 4096: 57 us with one wavefront per tile, 9 us with 16.
// ------------------------------------------------------------------------------------------
constexpr int kWgWaves = 16;
constexpr int kWgTiles = 160;      // W1 20 x 4 (80), W2 4 x 4 (16), W3 4 x 16 (64)
__global__ __launch_bounds__(64 * kWgWaves) void k_mlp_wgrad(MlpArgs a) {
  __shared__ float s_part[kWgWaves][256];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = blockIdx.x;
  if (w >= kWgTiles) {
    // bias gradients and the loss: 64 columns of the tiles' partial sums
    const int v = (w - kWgTiles) * 64 + lane;
    const int64_t tiles = a.ldT / 16;
    float sum = 0.0f;
    if (v < kPart)
#pragma unroll 4
      for (int64_t t = wave; t < tiles; t += kWgWaves) sum += a.part[t * kPart + v];
    s_part[wave][lane] = sum;
    __syncthreads();
    if (wave != 0 || v >= kPart) return;
    sum = 0.0f;
#pragma unroll
    for (int i = 0; i < kWgWaves; ++i) sum += s_part[i][lane];
    if (v < kHid) a.grad[kOffB1 + v] = sum;
    else if (v < 2 * kHid) a.grad[kOffB2 + v - kHid] = sum;
    else if (v < kPart - 1) a.grad[kOffB3 + v - 2 * kHid] = sum;
    else *a.loss = sum;
    return;
  }
  const uint16_t *A, *B;
  int mi, no, out_w, off;
  if (w < 80) {
    mi = w / 4; no = w % 4; A = a.xT; B = a.dz1T; out_w = kHid; off = kOffW1;
  } else if (w < 96) {
    mi = (w - 80) / 4; no = (w - 80) % 4; A = a.h1T; B = a.dz2T; out_w = kHid; off = kOffW2;
  } else {
    mi = (w - 96) / 16; no = (w - 96) % 16; A = a.h2T; B = a.dz3T; out_w = kBins; off = kOffW3;
  }
  // K = points: lane l takes points 8(l/16) .. +7 of each 32-point step (ldT is a multiple
  // of 32, padding points are zero)
  const uint16_t* arow = A + (size_t)(16 * mi + r) * a.ldT + 8 * g;
  const uint16_t* brow = B + (size_t)(16 * no + r) * a.ldT + 8 * g;
  f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int64_t ks = 32 * wave; ks < a.ldT; ks += 32 * kWgWaves) {
    const bf16x8 av = __builtin_bit_cast(bf16x8, *reinterpret_cast<const bf16x8s*>(arow + ks));
    const bf16x8 bv = __builtin_bit_cast(bf16x8, *reinterpret_cast<const bf16x8s*>(brow + ks));
    acc = mfma32(av, bv, acc);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) s_part[wave][(4 * g + t) * 16 + r] = acc[t];
  __syncthreads();
  if (tid >= 256) return;
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < kWgWaves; ++i) sum += s_part[i][tid];
  a.grad[off + (16 * mi + (tid >> 4)) * out_w + 16 * no + (tid & 15)] = sum;
}

// ------------------------------------------------------------------------------------------
// Adam
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, float* __restrict__ m,
                                              float* __restrict__ v,
                                              const float* __restrict__ gr, int64_t n, float lr,
                                              float b1, float b2, float eps, float ic1,
                                              float ic2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float g = gr[i];
  const float mi = b1 * m[i] + (1.0f - b1) * g;
  const float vi = b2 * v[i] + (1.0f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * ic1) / (sqrtf(vi * ic2) + eps);
}

// ------------------------------------------------------------------------------------------
hipError_t launch_mlp_frags(const float* params, uint16_t* frags, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_frags, dim3((kFrags * kFragElems + 255) / 256), dim3(256), 0, s,
                     params, frags);
  return hipGetLastError();
}

size_t mlp_frag_bytes() { return (size_t)kFrags * kFragElems * sizeof(uint16_t); }

hipError_t launch_mlp_infer(const MlpArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const int64_t tiles = (a.n + 15) / 16;
  hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_train(const MlpArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const int64_t tiles = a.ldT / 16;
  hipLaunchKernelGGL(k_mlp_train, dim3((unsigned)tiles), dim3(64 * kTrainWaves), 0, s, a);
  // the weight tiles, then 64 columns of bias/loss sums each
  hipLaunchKernelGGL(k_mlp_wgrad, dim3(kWgTiles + (kPart + 63) / 64), dim3(64 * kWgWaves), 0, s,
                     a);
  return hipGetLastError();
}

hipError_t launch_adam(float* p, float* m, float* v, const float* g, int64_t n, float lr,
                       float b1, float b2, float eps, float ic1, float ic2, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, m, v, g, n,
                     lr, b1, b2, eps, ic1, ic2);
  return hipGetLastError();
}

}  // namespace sopk
