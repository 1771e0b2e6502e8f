// The learned proposal's network outside the sampler: a forward pass in the
// sampler's precision (same device code) and the training step.
//
// Training minimises the mean over rows of -log q_re(t_re) - log q_im(t_im),
// where q_p is the learned proposal of one axis of one antenna: the
// discretised Gaussian over the levels j = 0..Q-1 with natural-log logits
// -kl (j - ml)^2, ml = mu_p + D_p, kl = kappa 2^clamp(b_p, -4, 4), (D_re, D_im,
// b_re, b_im) = network(features).  Derivatives of one axis' term:
//   d/d ml = -2 kl (t - E_q[j]),   d/d kl = (t - ml)^2 - E_q[(j - ml)^2],
//   d/d b  = kl ln 2 * d/d kl inside the clamp, 0 outside.
// The training network is float32 without rounding.  Two kernels:
//   grad:    every wavefront takes tiles of 16 rows through the forward pass, the loss, the
//            backward pass and the weight gradients dW = sum_r delta_r a_r^T on the float32
//            matrix cores, the sums kept in registers; one partial gradient per workgroup;
//   adam:    sums the partial gradients in a fixed order and updates the parameters and the
//            two moment estimates (Adam, Kingma & Ba).
// No atomics: the result does not depend on scheduling.
#include <cmath>

#include "../../include/dmala.h"
#include "common.hpp"
#include "host.hpp"
#include "mlp_device.hpp"

namespace dmala {

static_assert(kMlpParams == DMALA_MLP_PARAMS, "parameter count");
static_assert(kTrainRow == DMALA_TRAIN_ROW, "training row size");

// --------------------------------------------------------------- inference

__global__ __launch_bounds__(256) void mlp_forward_kernel(const float* __restrict__ w, const float* __restrict__ rows,
                                                          int n, int stride, float* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  mlp_stage<false>(w, lds);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = ((int64_t)blockIdx.x * 4 + wave) * 64 + (lane >> 4) * 16 + (lane & 15);
  float f[kMlpIn];
#pragma unroll
  for (int i = 0; i < kMlpIn; ++i) f[i] = row < n ? rows[(size_t)row * stride + i] : 0.f;
  const mlp_f32x4 o = mlp_eval4<false>(lds, 0u, mlp_inputs(f[0], f[1], f[2], f[3], f[4], f[5], f[6]));
  if (row < n) {
#pragma unroll
    for (int i = 0; i < kMlpOut; ++i) out[(size_t)row * kMlpOut + i] = o[i];
  }
}

// --------------------------------------------------------------- training

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTrainTile = 16;    // rows per wavefront tile
constexpr int kTrainWaves = 4;    // wavefronts per workgroup of the gradient kernel
constexpr int kTrainWgs = 256;    // its largest grid: one workgroup per CU, one wavefront per SIMD
constexpr int kPart = 4992;       // floats of one workgroup's partial gradient (4932 parameters, loss, pad)
static_assert(kMlpParams + 1 <= kPart, "partial record");
constexpr int kW2Ld = 68;         // LDS row stride of W2 and of the transposed tiles: 16 B reads of 4 columns and
                                  // 4 B reads of 16 columns x 4 rows each touch every bank once

// Tiles of n rows (any n of 32 bits: nothing here may pass 2^31).
__host__ __device__ inline int train_tiles(int n) { return n / kTrainTile + (n % kTrainTile != 0); }
// Workgroups of the gradient kernel for n rows (also the number of partial gradients).
inline int train_wgs(int n) {
  const int tiles = train_tiles(n), wgs = (tiles + kTrainWaves - 1) / kTrainWaves;
  return wgs < kTrainWgs ? wgs : kTrainWgs;
}

// Hidden units are numbered by their place in the tiles: place 16 t + 4 q + j is unit 16 t + 4 j + q (its own
// inverse), so that the K steps of the products below take the units in ascending order (see mlp_grad_kernel).
__host__ __device__ constexpr int hid_unit(int place) { return (place & ~15) | ((place & 3) << 2) | ((place >> 2) & 3); }

// Accumulators of one wavefront: the weight gradients as 16 x 16 tiles (register j of lane (q, c), q = lane / 16,
// c = lane % 16: row 4 q + j, column c), b2's as per-lane sums over the lane's rows, b3's and the loss.
struct GradAcc {
  f32x4 g2[4][4], g1[4], g3[4], b2[4], b3;
  float loss;
};
constexpr int kAccRegs = 16 * 4 + 3 * 16 + 4 + 1;

// every accumulator register v, numbered, becomes f(number, v)
template <typename F>
__device__ __forceinline__ void for_acc(GradAcc& a, F&& f) {
  int i = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int u = 0; u < 4; ++u) a.g2[t][u][j] = f(i++, a.g2[t][u][j]);
      a.g1[t][j] = f(i++, a.g1[t][j]);
      a.g3[t][j] = f(i++, a.g3[t][j]);
      a.b2[t][j] = f(i++, a.b2[t][j]);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) a.b3[j] = f(i++, a.b3[j]);
  a.loss = f(i++, a.loss);
}

// Loss, forward, backward and weight gradients of the rows, all on the float32 matrix cores
// (v_mfma_f32_16x16x4f32: A (16 x 4) lane l holds A[l % 16][l / 16], B (4 x 16) lane l holds B[l / 16][l % 16],
// register j of the accumulator D[4 (l / 16) + j][l % 16]).  A wavefront takes 16 rows at a time as the columns of
// every product: lane (q, c) then holds the hidden units in places 16 t + 4 q + j of row c, and the next layer's K
// step (t, j) uses exactly those registers as its B operand (weights read in that K order), so that forward and
// backward exchange nothing between lanes.
// A unit whose input is within rounding of zero is on or off by the order of its sum, and one such unit of a
// batch's millions moves the gradient by more than all other rounding (65 536 rows: 3e-6 against 3e-7 of the 2-norm).
// The order is therefore fixed: the bias first, then fused multiply-adds over ascending inputs.  The matrix core
// does its K terms as that chain (ascending k from the accumulator, one rounding each), and with the units' places
// (hid_unit) K step (t, j) takes units 16 t + 4 j .. + 3, so that forward and backward sums are those of a loop over
// the units bit for bit.
// The weight gradients contract over the rows; their operands are the transposed
// tiles, which pass through LDS (two 16 x 64 tiles per wavefront).  236 products per tile, 8 passes each: the
// products of 65 536 rows need 13 us at the float32 matrix rate.  Measured 39-41 us (40 % of a wave's cycles in
// products, 35 % waiting on LDS and on dependent products with one wavefront per SIMD, which the 117 accumulator
// registers ask for); nothing per row goes to memory: one thread per row that wrote its activations out, and a
// second kernel that read them back for the weight gradients, took 140 us.
__global__ __launch_bounds__(64 * kTrainWaves) __attribute__((amdgpu_waves_per_eu(1, 1)))
void mlp_grad_kernel(const float* __restrict__ w, const float* __restrict__ rows, const int32_t* __restrict__ tgt,
                     int n, float inv_n, float* __restrict__ part) {
  // W2, then per wavefront two transposed tiles, the inputs and the output gradients; reused for the
  // sum over the workgroup's wavefronts
  constexpr int kWaveLds = 2 * kTrainTile * kW2Ld + kTrainTile * 8 + kTrainTile * 4;
  constexpr int kLds = kMlpHid * kW2Ld + kTrainWaves * kWaveLds;
  constexpr int kSlots = 2 * kAccRegs * 64;
  __shared__ __attribute__((aligned(16))) float lds[kLds > kSlots ? kLds : kSlots];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, q = lane >> 4;
  float* W2 = lds;
  float* bufA = lds + kMlpHid * kW2Ld + wave * kWaveLds;
  float* bufB = bufA + kTrainTile * kW2Ld;
  float* xs = bufB + kTrainTile * kW2Ld;
  float* ds = xs + kTrainTile * 8;
  // (rows and columns by place)
  for (int i = tid; i < kMlpHid * kMlpHid; i += 64 * kTrainWaves)
    W2[hid_unit(i >> 6) * kW2Ld + hid_unit(i & 63)] = w[kOffW2 + i];
  // first-layer weights, [place 16 t + c][input 4 s + q] (input 7, the constant 1 of b1's gradient, with weight 0);
  // third layer in the K order of the lane's units, its 4 rows repeated in every group of 4 so that each lane group
  // gets all 4 outputs; and its transpose
  float w1[4][2], w3[4][4], w3t[4];
  f32x4 b1v[4], b2v[4], b3v;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int u = hid_unit(16 * t + c);
    w1[t][0] = w[kOffW1 + u * kMlpIn + q];
    w1[t][1] = q < 3 ? w[kOffW1 + u * kMlpIn + 4 + q] : 0.f;
    w3t[t] = w[kOffW3 + q * kMlpHid + u];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = hid_unit(16 * t + 4 * q + j);
      w3[t][j] = w[kOffW3 + (c & 3) * kMlpHid + v];
      b1v[t][j] = w[kOffB1 + v];
      b2v[t][j] = w[kOffB2 + v];
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) b3v[j] = w[kOffB3 + j];
  __syncthreads();
  GradAcc acc;
  for_acc(acc, [](int, float) { return 0.f; });

  const int tiles = train_tiles(n);
  // the lane's part of a row: inputs q and 4 + q, and the centre, precision, level count and target of axis q % 2
  struct RowIn { float x0, x1, mu, kap, qf; int t; };
  auto load_row = [&](int tile) {
    const int64_t r = (int64_t)tile * kTrainTile + c;   // (tiles past the end: past 2^31 where n is near it)
    const bool ok = r < n;
    const float* row = rows + (size_t)(ok ? r : 0) * kTrainRow;
    RowIn v;
    v.x0 = row[q]; v.x1 = row[4 + q]; v.mu = row[7 + (q & 1)]; v.kap = row[9]; v.qf = row[10];
    v.t = tgt[2 * (size_t)(ok ? r : 0) + (q & 1)];
    if (!ok) v = RowIn{0.f, 0.f, 0.f, 1.f, 2.f, 0};
    if (q == 3) v.x1 = 1.f;
    return v;
  };
  RowIn next = load_row(blockIdx.x * kTrainWaves + wave);
  for (int tile = blockIdx.x * kTrainWaves + wave; tile < tiles; tile += gridDim.x * kTrainWaves) {
    const bool ok = tile * kTrainTile + c < n;
    const float x0 = next.x0, x1 = next.x1, mup = next.mu, kap = next.kap, qf = next.qf;
    const int tg = next.t;
    next = load_row(tile + gridDim.x * kTrainWaves);   // in flight during this tile (past the end: row 0, unused)
    // forward
    f32x4 a1[4], a2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[t][0], x0, b1v[t], 0, 0, 0);
      z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[t][1], x1, z, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) a1[t][j] = fmaxf(z[j], 0.f);
      a2[t] = b2v[t];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      f32x4 av[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) av[t] = *(const f32x4*)(W2 + (16 * t + c) * kW2Ld + 16 * s + 4 * q);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t) a2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t][j], a1[s][j], a2[t], 0, 0, 0);
    }
    f32x4 out = b3v;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a2[s][j] = fmaxf(a2[s][j], 0.f);
        out = __builtin_amdgcn_mfma_f32_16x16x4f32(w3[s][j], a2[s][j], out, 0, 0, 0);
      }
    // loss and its gradient with respect to the outputs: lane group q takes axis q % 2 of its row
    const int Q = qf >= 16.f ? 16 : (qf >= 2.f ? (int)qf : 2);
    const bool im = q & 1;
    const float oD = im ? out[1] : out[0], ob = im ? out[3] : out[2];
    const float ml = mup + oD, kl = kap * exp2f(fminf(fmaxf(ob, -4.f), 4.f));
    // the largest logit is the nearest level's, or with a negative precision the farthest one's; lane groups q and
    // q ^ 2 share an axis and take half its levels each
    const float top = (float)(Q - 1);
    const float d0 = (kl < 0.f ? (ml + ml > top ? 0.f : top) : fminf(fmaxf(rintf(ml), 0.f), top)) - ml;
    const float mx = -kl * d0 * d0;
    float Z = 0.f, Ej = 0.f, Ed2 = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int j = 2 * i + (q >> 1);
      const float d = j - ml;
      const float e = j < Q ? expf(-kl * d * d - mx) : 0.f;
      Z += e; Ej += e * j; Ed2 += e * d * d;
      if (i == 3 && !__any(Q > 8)) break;
    }
    Z += __shfl_xor(Z, 32); Ej += __shfl_xor(Ej, 32); Ed2 += __shfl_xor(Ed2, 32);
    Ej /= Z; Ed2 /= Z;
    const float dt = tg - ml;
    const float sc = ok ? inv_n : 0.f;
    float ls = kl * dt * dt + mx + logf(Z);
    float dD = -2.f * kl * (tg - Ej);
    float db = (fabsf(ob) < 4.f) ? (dt * dt - Ed2) * kl * 0.69314718055994531f : 0.f;
    ls = ok ? ls * sc : 0.f;
    dD = ok ? dD * sc : 0.f;
    db = ok ? db * sc : 0.f;
    const float pD = __shfl_xor(dD, 16), pb = __shfl_xor(db, 16);
    const f32x4 dout = {im ? pD : dD, im ? dD : pD, im ? pb : db, im ? db : pb};
    if (q < 2) acc.loss += ls;
    if (q == 0) acc.b3 += dout;
    // backward to the hidden layers
    f32x4 d1[4], d2[4];
    const float dq = q == 0 ? dout[0] : (q == 1 ? dout[1] : (q == 2 ? dout[2] : dout[3]));
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      d2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w3t[t], dq, z, 0, 0, 0);
      d1[t] = z;
#pragma unroll
      for (int j = 0; j < 4; ++j) d2[t][j] = a2[t][j] > 0.f ? d2[t][j] : 0.f;
      acc.b2[t] += d2[t];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float* wr = W2 + (16 * s + 4 * q + j) * kW2Ld + c;
#pragma unroll
        for (int t = 0; t < 4; ++t) d1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[16 * t], d2[s][j], d1[t], 0, 0, 0);
      }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) d1[t][j] = a1[t][j] > 0.f ? d1[t][j] : 0.f;
    // weight gradients: the tiles transposed to [row][unit] (LDS of this wavefront alone: its own order suffices)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      *(f32x4*)(bufA + c * kW2Ld + 16 * t + 4 * q) = a1[t];
      *(f32x4*)(bufB + c * kW2Ld + 16 * t + 4 * q) = d2[t];
    }
    xs[c * 8 + q] = x0;
    xs[c * 8 + 4 + q] = x1;
    if (q == 0) *(f32x4*)(ds + c * 4) = dout;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float av[4], dv[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        av[t] = bufA[(4 * s + q) * kW2Ld + 16 * t + c];
        dv[t] = bufB[(4 * s + q) * kW2Ld + 16 * t + c];
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc.g2[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[t], av[u], acc.g2[t][u], 0, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      *(f32x4*)(bufA + c * kW2Ld + 16 * t + 4 * q) = a2[t];
      *(f32x4*)(bufB + c * kW2Ld + 16 * t + 4 * q) = d1[t];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float av[4], dv[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        av[t] = bufA[(4 * s + q) * kW2Ld + 16 * t + c];
        dv[t] = bufB[(4 * s + q) * kW2Ld + 16 * t + c];
      }
      const float xv = c < 8 ? xs[(4 * s + q) * 8 + (c & 7)] : 0.f;
      const float ov = c < kMlpOut ? ds[(4 * s + q) * 4 + (c & 3)] : 0.f;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        acc.g1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[t], xv, acc.g1[t], 0, 0, 0);
        acc.g3[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ov, av[t], acc.g3[t], 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // sum over the wavefronts in a fixed order, (0 + 2) + (1 + 3), through two register-image slots
  __syncthreads();
  float* slot = lds + (wave & 1) * kAccRegs * 64 + lane;
  if (wave >= 2) for_acc(acc, [&](int i, float v) { return slot[i * 64] = v; });
  __syncthreads();
  if (wave < 2) for_acc(acc, [&](int i, float v) { return v + slot[i * 64]; });
  __syncthreads();
  if (wave == 1) for_acc(acc, [&](int i, float v) { return slot[i * 64] = v; });
  __syncthreads();
  if (wave != 0) return;
  slot += kAccRegs * 64;
  for_acc(acc, [&](int i, float v) { return v + slot[i * 64]; });
  // b2 and b3 over the 16 rows of a tile's lanes, the loss over all lanes
#pragma unroll
  for (int s = 1; s < 16; s <<= 1) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int t = 0; t < 4; ++t) acc.b2[t][j] += __shfl_xor(acc.b2[t][j], s);
      acc.b3[j] += __shfl_xor(acc.b3[j], s);
    }
    acc.loss += __shfl_xor(acc.loss, s);
  }
  acc.loss += __shfl_xor(acc.loss, 16);
  float* out = part + (size_t)blockIdx.x * kPart;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int u = hid_unit(16 * t + 4 * q + j);
#pragma unroll
      for (int i = 0; i < 4; ++i) out[kOffW2 + u * kMlpHid + hid_unit(16 * i + c)] = acc.g2[t][i][j];
      if (c < kMlpIn) out[kOffW1 + u * kMlpIn + c] = acc.g1[t][j];
      if (c == kMlpIn) out[kOffB1 + u] = acc.g1[t][j];
      if (c == 0) out[kOffB2 + u] = acc.b2[t][j];
      if (q == 0) out[kOffW3 + j * kMlpHid + hid_unit(16 * t + c)] = acc.g3[t][j];
    }
    if (lane == 0) out[kOffB3 + j] = acc.b3[j];
  }
  if (lane == 0) out[kMlpParams] = acc.loss;
}

// Adam on 64 parameters per workgroup.  Its 8 wavefronts each sum every eighth partial gradient (the sums then
// meet in LDS in a fixed order): with one thread per parameter alone, the 256 dependent trips to the partials took
// 63 us; 78 workgroups x 8 slices with 8 loads in flight are bound by the latency of 4 trips.
constexpr int kAdamSlices = 8;
__global__ __launch_bounds__(64 * kAdamSlices) void mlp_adam_kernel(float* __restrict__ w, float* __restrict__ m,
                                                                    float* __restrict__ v, const float* __restrict__ part,
                                                                    int chunks, int step, float lr, float* __restrict__ loss,
                                                                    float* __restrict__ grad) {
  __shared__ float sums[kAdamSlices][64];
  const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
  float g = 0.f;
  const float* src = part + (size_t)sl * kPart + p;
#pragma unroll 8
  for (int k = sl; k < chunks; k += kAdamSlices) {
    g += *src;
    src += (size_t)kAdamSlices * kPart;
  }
  sums[sl][lane] = g;
  __syncthreads();
  if (sl != 0 || p > kMlpParams) return;
#pragma unroll
  for (int k = 1; k < kAdamSlices; ++k) g += sums[k][lane];
  if (p == kMlpParams) {
    if (loss) loss[0] = g;
    return;
  }
  if (grad) grad[p] = g;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float mn = b1 * m[p] + (1.f - b1) * g;
  const float vn = b2 * v[p] + (1.f - b2) * g * g;
  m[p] = mn;
  v[p] = vn;
  const float mh = mn / (1.f - powf(b1, (float)step));
  const float vh = vn / (1.f - powf(b2, (float)step));
  w[p] -= lr * mh / (sqrtf(vh) + eps);
}

}  // namespace dmala

using namespace dmala;
using namespace dmala::host;

extern "C" {

dmala_status dmala_mlp_forward(const float* weights, const float* rows, int32_t n_rows, int32_t row_stride, float* out,
                               dmala_stream_t stream) {
  if (!weights || !rows || !out) return fail(DMALA_ERR_ARG, "weights, rows and out must be non-NULL");
  if (n_rows < 0) return fail(DMALA_ERR_ARG, "n_rows must be >= 0");
  if (row_stride < kMlpIn) return fail(DMALA_ERR_ARG, "row_stride must be >= %d", kMlpIn);
  if (n_rows == 0) return DMALA_OK;
  const int blocks = n_rows / 256 + (n_rows % 256 != 0);
  hipLaunchKernelGGL(mlp_forward_kernel, dim3(blocks), dim3(256), mlp_lds_bytes<false>(), (hipStream_t)stream, weights, rows,
                     n_rows, row_stride, out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mlp forward launch");
  g_err.clear();
  return DMALA_OK;
}

size_t dmala_mlp_train_workspace_size(int32_t n_rows) {
  if (n_rows < 1) return 0;
  return round_up((size_t)train_wgs(n_rows) * kPart * sizeof(float), 256);
}

dmala_status dmala_mlp_train_step(float* weights, float* adam_m, float* adam_v, int32_t step, float lr,
                                  const float* rows, const int32_t* targets, int32_t n_rows, float* loss, float* grad,
                                  void* workspace, size_t workspace_bytes, dmala_stream_t stream) {
  if (!weights || !adam_m || !adam_v || !rows || !targets) return fail(DMALA_ERR_ARG, "NULL argument");
  if (n_rows < 1) return fail(DMALA_ERR_ARG, "n_rows must be >= 1");
  if (step < 1) return fail(DMALA_ERR_ARG, "step counts from 1");
  if (!(lr > 0.f) || !std::isfinite(lr)) return fail(DMALA_ERR_ARG, "lr must be positive and finite");
  if (!workspace) return fail(DMALA_ERR_WORKSPACE, "workspace is NULL");
  const size_t need = dmala_mlp_train_workspace_size(n_rows);
  if (workspace_bytes < need) return fail(DMALA_ERR_WORKSPACE, "workspace too small: %zu < %zu bytes", workspace_bytes, need);
  if (((uintptr_t)workspace & 255) != 0) return fail(DMALA_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  float* part = (float*)workspace;
  const int wgs = train_wgs(n_rows);
  hipLaunchKernelGGL(mlp_grad_kernel, dim3(wgs), dim3(64 * kTrainWaves), 0, s, weights, rows, targets, n_rows,
                     1.0f / (float)n_rows, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mlp gradient launch");
  hipLaunchKernelGGL(mlp_adam_kernel, dim3((kMlpParams + 1 + 63) / 64), dim3(64 * kAdamSlices), 0, s, weights, adam_m, adam_v,
                     part, wgs, step, lr, loss, grad);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "mlp adam launch");
  g_err.clear();
  return DMALA_OK;
}

}  // extern "C"
