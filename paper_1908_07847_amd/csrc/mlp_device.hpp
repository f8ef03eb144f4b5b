// Device-side helpers shared by the libmlp kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mlp.h"

namespace mlpk {

constexpr int kWave = 64;
constexpr int kLayerMaxOut = 16;  // outputs supported by the generic layer kernels

// Logistic sigmoid (Equation 1) from the hardware base-2 exponential and
// reciprocal.  e^-z = 2^(-z log2 e).  Published methods used:
//  - log2 e held as a two-part constant, a high part plus its tail, in the
//    manner of Cody and Waite's argument reduction (Cody & Waite, "Software
//    Manual for the Elementary Functions", 1980);
//  - the rounding error of the product -z * L_HI obtained exactly with one
//    FMA, the error-free transformation TwoProductFMA (Ogita, Rump & Oishi,
//    "Accurate sum and dot product", SIAM J. Sci. Comput. 2005);
//  - 2^(th + tl) = 2^th (1 + tl ln 2) to first order in the small tail tl;
//  - one Newton-Raphson iteration r <- r + r (1 - d r) on the hardware
//    reciprocal of d = 1 + e^-z.
// The exponent so keeps ~48 bits and the result is within a few float ulps
// of the exact sigmoid (checked against float64 in the tests).  For
// z < -87 the exponent is clamped at 2^126 (sigma ~ 1e-38 instead of 0).
__device__ __forceinline__ float sigmoid_e(float z, float &e_out) {
  const float L_HI = 1.44269502162933349609375f;    // float(log2 e)
  const float L_LO = 1.925963033500011079e-08f;     // log2 e - L_HI
  const float LN2 = 0.693147180559945309f;
  float th = -z * L_HI;
  float err = fmaf(-z, L_HI, -th);
  float tl = fmaf(-z, L_LO, err);
  th = fminf(th, 126.0f);
  float e = __builtin_amdgcn_exp2f(th);
  e = fmaf(e, tl * LN2, e);
  float d = 1.0f + e;
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(r, fmaf(-d, r, 1.0f), r);
  e_out = e;
  return r;
}

// sigma and its slope from e = e^-z as sigmoid_e left it: the same bits as
// sigmoid_slope(z) without the exponential.
__device__ __forceinline__ float sigmoid_slope_of_e(float e, float &slope) {
  const float d = 1.0f + e;
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(r, fmaf(-d, r, 1.0f), r);
  slope = (e * r) * r;
  return r;
}

// sigmoid_e of four values, stage by stage: the same bits; left to itself the
// compiler may run the four chains one after the other (60 cycles each).
__device__ __forceinline__ void sigmoid_e4(const float *z, float *a, float *e) {
  const float L_HI = 1.44269502162933349609375f, L_LO = 1.925963033500011079e-08f, LN2 = 0.693147180559945309f;
  float tl[4], r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float th = -z[i] * L_HI;
    tl[i] = fmaf(-z[i], L_LO, fmaf(-z[i], L_HI, -th)) * LN2;
    e[i] = __builtin_amdgcn_exp2f(fminf(th, 126.0f));
  }
  asm volatile("" : "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    e[i] = fmaf(e[i], tl[i], e[i]);
    a[i] = 1.0f + e[i];
    r[i] = __builtin_amdgcn_rcpf(a[i]);
  }
  asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = fmaf(r[i], fmaf(-a[i], r[i], 1.0f), r[i]);
}

__device__ __forceinline__ float sigmoid(float z) {
  float e;
  return sigmoid_e(z, e);
}

// sigma(z) and its slope sigma(z) (1 - sigma(z)) = e^-z sigma(z)^2.  The
// second form keeps full relative precision where sigma is close to 1 (there
// 1 - sigma would cancel); for z < -87 it underflows to 0 instead of ~1e-38.
__device__ __forceinline__ float sigmoid_slope(float z, float &slope) {
  float e;
  const float a = sigmoid_e(z, e);
  slope = (e * a) * a;
  return a;
}

// The tanh hidden activation (a variant; the paper's neurons are sigmoid)
// and its slope 1 - tanh(z)^2.
__device__ __forceinline__ float tanh_slope(float z, float &slope) {
  const float a = tanhf(z);
  slope = 1.0f - a * a;
  return a;
}

// Hidden activation by kind (0: sigma, 1: tanh) and its slope.
__device__ __forceinline__ float hidden_act(int act, float z, float &slope) {
  return act == 1 ? tanh_slope(z, slope) : sigmoid_slope(z, slope);
}

// theta <- theta - lr*g.  With a compensation term c (Kahan summation of the
// update stream) the low-order bits lost when a small step is added to a
// larger weight are carried to the next update instead of being dropped.
__device__ __forceinline__ void gd_update(float &w, float &c, float lr, float g, bool compensated) {
  if (compensated) {
    float y = -lr * g - c;
    float t = w + y;
    c = (t - w) - y;
    w = t;
  } else {
    w = w - lr * g;
  }
}

// Buffer loads: from a uniform base with a 32-bit byte offset; an offset past
// `bytes` reads zero, so a batch needs no masks and no 64-bit addresses.
// (Written with clamped 64-bit addresses, a batch of loads was issued one by
// one, each waited for, where scalar registers ran out.)
// Resources are under 2 GB, so kNoLoad plus an offset inside one stays past the end.
constexpr uint32_t kNoLoad = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gbuf(const float *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float gld(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

// Lanes 0..31: a plus a of lane + 32; lanes 32..63: b plus b of lane - 32 (one
// exchange in the vector unit; a shuffle goes through the LDS crossbar).
__device__ __forceinline__ float add_swap32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                  false, false);
  const uint32_t x = r[0], y = r[1];
  return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
}
// The same between neighbouring rows of 16 lanes: even rows a, odd rows b.
__device__ __forceinline__ float add_swap16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                  false, false);
  const uint32_t x = r[0], y = r[1];
  return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
}

// Sum over lanes l, l + 16, l + 32, l + 48, in every one of them.
__device__ __forceinline__ float sum_rows(float v) {
  v = add_swap16(v, v);
  return add_swap32(v, v);
}

// v plus lane (v) permuted by a DPP row pattern (a VALU op, no LDS traffic).
template <int CTRL>
__device__ __forceinline__ float add_dpp(float v) {
  const int s = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false);
  return v + __builtin_bit_cast(float, s);
}

// Sum over the 64 lanes of a wave, fixed butterfly order (deterministic).
__device__ __forceinline__ float wave_sum(float v) {
  v = add_swap32(v, v);
  v = add_swap16(v, v);
  v = add_dpp<0x128>(v);   // row_ror 8
  v += __shfl_xor(v, 4, kWave);
  v = add_dpp<0x4E>(v);    // quad_perm [2,3,0,1]
  return add_dpp<0xB1>(v); // quad_perm [1,0,3,2]
}

__device__ __forceinline__ int round_up(int v, int m) { return (v + m - 1) / m * m; }

// Sum over each row of 16 lanes: swap neighbours, swap pairs, mirror within
// 8, mirror within 16.  Every lane of the row ends with the same value
// (each step adds two equal-order partial sums), so the result is bitwise
// identical across the row and across runs.
__device__ __forceinline__ float sum16(float v) {
  v = add_dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v = add_dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v = add_dpp<0x141>(v);  // row_half_mirror
  v = add_dpp<0x140>(v);  // row_mirror
  return v;
}

}  // namespace mlpk

// Launch wrappers implemented in the .hip files and used by the host API.
namespace mlph {

// Rows whose deltas the backward workspace could hold: its size, min(n, this)
// (H + K + 1) floats, bounds the partial gradients of the row ranges.
constexpr int64_t kBackwardChunk = 16384;

// Small-network trainer: one workgroup per net, all epochs in one launch.
// items == nullptr means a single net described by `one`.  threads is 128,
// 256 or 512 (waves split the rows), or kHiddenSplit: one wave per 16
// hidden units of the widest net (waves split the hidden layer; the paper's
// sigmoid network without momentum, others fall back to 128 threads).
// small_threads picks it from the net count, the widest net and a hint.
constexpr int kHiddenSplit = 64;
size_t small_lds_bytes(int n_rows, int n_hidden, int n_in, int threads, bool momentum = false);
size_t small_launch_lds_bytes(int max_rows, int max_hidden, int n_in, int threads, bool momentum = false);
int small_threads(int n_nets, int max_hidden, int n_cu, int hint);
// act: hidden activation (0 sigma, 1 tanh); vel != nullptr: heavy-ball
// momentum mu with the velocity vel[P] (packed, a single net only).
hipError_t launch_small_train(const mlp_batch_item *items, mlp_batch_item one, int n_nets,
                              int n_in, int n_out, int max_rows, int max_hidden, const float *X,
                              const float *T, float *theta, float *comp, int epochs,
                              float *loss_hist, int act, float mu, float *vel, int threads, hipStream_t s);

// Generic layer kernels (any sizes) for mlp_forward / mlp_backward / mlp_step.
hipError_t launch_forward(int64_t n, int D, int H, int K, const float *X, mlp_params p, float *A,
                          float *Y, int act, int n_cu, hipStream_t s);
hipError_t launch_backward(int64_t n, int64_t ws_floats, int D, int H, int K, const float *X,
                           const float *A, const float *Y, const float *dY, const float *T,
                           mlp_params p, mlp_params g, float *dX, float *loss, float *ws, int act,
                           hipStream_t s);
hipError_t launch_step(int D, int H, int K, mlp_params p, mlp_params g, float *comp, float lr, float mu,
                       float *vel, hipStream_t s);
hipError_t launch_predict(int64_t n, int D, int H, int K, const float *X, mlp_params p, float *Y,
                          int32_t *labels, const float *T, int32_t *correct, int act, int n_cu, hipStream_t s);
// One dense layer (several-hidden-layer networks) and a packed update.
hipError_t launch_dense_forward(int64_t n, int din, int dout, const float *X, const float *W, const float *b,
                                int act, float *Y, hipStream_t s);
hipError_t launch_dense_backward(int64_t n, int din, int dout, const float *X, const float *Y, const float *dY,
                                 const float *W, int act, float *gW, float *gb, float *dX, float *ws,
                                 hipStream_t s);
hipError_t launch_update(int64_t P, float *theta, const float *g, float *comp, float lr, hipStream_t s);
hipError_t launch_mse_grad(int64_t n, int k, const float *Y, const float *T, float *dY, float *loss, hipStream_t s);
hipError_t launch_eval_batched(const mlp_batch_item *items_dev, int n_nets, int max_rows, int max_hidden, int D, int K,
                               const float *X, const float *T, const float *theta, float *loss, int32_t *correct,
                               hipStream_t s);
hipError_t launch_cv_select(const float *loss, const int32_t *group, int n_nets, int n_groups, float *group_mean,
                            int32_t *best, hipStream_t s);

}  // namespace mlph
