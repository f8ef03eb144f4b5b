// Separate forward / backward / update kernels (arxiv 1908.07847,
// section 2.2), for callers that drive the steps themselves -- e.g. a
// torch.autograd.Function whose backward is this hand-written adjoint.
//
//  k_forward_rows  n_in <= 64, n_out <= 4: W1 in LDS once per workgroup, rows
//                  straight from memory to the operands, a wave walking its
//                  16-row sets; predictions take class and count from the
//                  outputs in registers
//  k_forward_tiled 64 rows per workgroup, 16 per wave: the row tile of X and
//                  a 64-unit block of W1 at a time in LDS, z1 on
//                  v_mfma_f32_16x16x4_f32, sigma in the accumulator layout,
//                  the output layer as lane partials summed across the 16
//                  lanes of a row (n_in <= 256, n_out <= 16)
//  k_forward       one thread per row (any n_in): z1 = X W1^T + b1,
//                  A = sigma(z1), Y = sigma(A W2^T + b2).
//  backward        grad.hpp: the output deltas (dY from the caller, or the MSE
//                  reading 2 (Y - T) / (n K)) and delta1 = (delta2 W2) .
//                  A (1 - A) are formed where the gradient sums and the
//                  optional dX = delta1 W1 consume them; row sums run in
//                  a fixed order, so the result is bitwise repeatable.
//  k_step          theta <- theta - lr g, optionally Kahan-compensated; with
//                  a velocity buffer, heavy-ball momentum (v <- mu v + g,
//                  theta <- theta - lr v).  Forward and backward take the
//                  hidden activation (sigma, or the tanh variant).
//  k_eval_tiled    one workgroup per net of a batched item table, z1 on the
//                  matrix cores, hidden tiles over the waves; k_eval_rows rows
//                  over the waves, for nets of up to 16 units; k_cv_means,
//                  k_cv_best: the folds' mean losses and the best group
//  k_eval_batched  the same for any n_in, n_out: loss and
//                  correct count of the net on its own rows (e.g. a held-out
//                  fold), threads over rows, fixed-order block sums
//  k_argmax        rows in a grid-stride loop (at most 512 workgroups): the
//                  class is the index of the largest
//                  output (lowest index on ties); with one-hot targets, the
//                  count of rows whose class matches the target's, summed
//                  per block and added once per block (integer adds, so the
//                  count does not depend on their order).
#include <algorithm>

#include "grad.hpp"
#include "mlp_device.hpp"

namespace mlpk {

__global__ __launch_bounds__(256) void k_forward(int64_t n, int D, int H, int K,
                                                 const float *__restrict__ X, mlp_params p,
                                                 float *__restrict__ A, float *__restrict__ Y, int act) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const float *x = X + r * D;
  float z2[kLayerMaxOut];
  for (int k = 0; k < K && k < kLayerMaxOut; ++k) z2[k] = p.b2[k];
  for (int h = 0; h < H; ++h) {
    const float *w = p.W1 + (int64_t)h * D;
    float z = p.b1[h];
    for (int d = 0; d < D; ++d) z += x[d] * w[d];
    float slope;
    const float a = hidden_act(act, z, slope);
    if (A) A[r * H + h] = a;
    for (int k = 0; k < K && k < kLayerMaxOut; ++k) z2[k] += a * p.W2[(int64_t)k * H + h];
  }
  for (int k = 0; k < K && k < kLayerMaxOut; ++k) Y[r * K + k] = sigmoid(z2[k]);
}

constexpr int kFwdRows = 64, kFwdHB = 64, kFwdMaxD = 256;

typedef float f32x4_l __attribute__((ext_vector_type(4)));

// KO: output slots held per row in registers (K <= KO); ACT: the hidden
// activation (0 sigma, 1 tanh).
template <int KO, int ACT>
__global__ __launch_bounds__(256) void k_forward_tiled(int64_t n, int D, int H, int K,
                                                       const float *__restrict__ X, mlp_params p,
                                                       float *__restrict__ A, float *__restrict__ Y) {
  extern __shared__ float4 fsm4[];
  float *sm = reinterpret_cast<float *>(fsm4);
  const int DK = (D + 3) / 4 * 4, XS = DK + 1;     // contraction length; odd row stride
  float *xs = sm;                                   // [64][XS]
  float *ws = xs + kFwdRows * XS;                   // [64][XS] W1 block
  float *w2 = ws + kFwdHB * XS;                     // [16][64] W2 block
  float *b1 = w2 + kLayerMaxOut * kFwdHB;           // [64]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kFwdRows;
  const int rows = (int)min((int64_t)kFwdRows, n - r0);
  for (int q = tid; q < kFwdRows * XS; q += 256) {
    const int r = q / XS, c = q - r * XS;
    xs[q] = (r < rows && c < D) ? X[(r0 + r) * D + c] : 0.0f;
  }
  float zp[4][KO];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int k = 0; k < KO; ++k) zp[i][k] = 0.0f;
  for (int h0 = 0; h0 < H; h0 += kFwdHB) {
    __syncthreads();   // the previous block's W1 / W2 are no longer read
    for (int q = tid; q < kFwdHB * XS; q += 256) {
      const int h = q / XS, c = q - h * XS;
      ws[q] = (h0 + h < H && c < D) ? p.W1[(int64_t)(h0 + h) * D + c] : 0.0f;
    }
    for (int q = tid; q < kLayerMaxOut * kFwdHB; q += 256) {
      const int k = q / kFwdHB, h = q - k * kFwdHB;
      w2[q] = (k < K && h0 + h < H) ? p.W2[(int64_t)k * H + h0 + h] : 0.0f;
    }
    if (tid < kFwdHB) b1[tid] = h0 + tid < H ? p.b1[h0 + tid] : 0.0f;
    __syncthreads();
    for (int ht = 0; ht < kFwdHB / 16; ++ht) {
      if (h0 + ht * 16 >= H) break;
      f32x4_l z = {0.f, 0.f, 0.f, 0.f};
      const float *xa = xs + (wave * 16 + l16) * XS + lg;
      const float *wb = ws + (ht * 16 + l16) * XS + lg;
      for (int k0 = 0; k0 < DK; k0 += 4) z = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[k0], wb[k0], z, 0, 0, 0);
      const int hl = ht * 16 + l16, h = h0 + hl;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = wave * 16 + 4 * lg + i;
        float slope;
        const float a = h < H ? hidden_act(ACT, z[i] + b1[hl], slope) : 0.0f;
        if (A && r < rows && h < H) A[(r0 + r) * H + h] = a;
#pragma unroll
        for (int k = 0; k < KO; ++k)
          if (k < K) zp[i][k] = fmaf(a, w2[k * kFwdHB + hl], zp[i][k]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = wave * 16 + 4 * lg + i;
#pragma unroll
    for (int k = 0; k < KO; ++k) {
      if (k < K) {
        const float z2 = sum16(zp[i][k]);
        if (l16 == 0 && r < rows) Y[(r0 + r) * K + k] = sigmoid(z2 + p.b2[k]);
      }
    }
  }
}

// Class of a row of outputs (or targets): the largest entry, the lowest
// index on ties; a single output is a two-class net, class 1 above 1/2.
__device__ __forceinline__ int argmax_row(const float *v, int K) {
  if (K == 1) return v[0] > 0.5f ? 1 : 0;
  int best = 0;
  for (int k = 1; k < K; ++k)
    if (v[k] > v[best]) best = k;   // strict: the lowest index wins ties
  return best;
}

// Forward pass (and class predictions) for n_in <= 64 and at most 4 outputs.
// A workgroup of 4 waves walks the rows, 32 per wave at a time (two 16-row
// tiles that share every W1 operand and interleave their product chains):
// the X operands go from global memory into registers, W1 | b1 | W2 sit in
// LDS -- staged once per workgroup when the whole hidden layer fits kFwrHB
// units, else block by block.  After the last hidden tile, lane 4 i + k of a
// row group holds output k of row i, so one sigmoid per lane finishes four
// rows, and the class (and the count against targets) comes from the same
// registers.  The products, the activation and the output sums run in
// k_forward_tiled's order, so the outputs are the same bits.
// Bound: the float32 matrix cores (2 D H of the row's flops) and the vector
// ALU of the activation about equally; the next rows' X loads overlap.
// Staging X and W1 per 64 rows with an index division per element held
// 1,048,576 rows of a 33-256-3 network at 582 us with the separate argmax,
// now 341.
constexpr int kFwrHB = 256;

struct PredictOut {
  int32_t *labels;     // null: forward pass only
  const float *T;      // null: no count
  int32_t *correct;
};

__device__ __forceinline__ float quad_bcast(float v, int k) {
  const int b = __builtin_bit_cast(int, v);
  const int r = k == 0 ? __builtin_amdgcn_update_dpp(0, b, 0x00, 0xF, 0xF, false)
              : k == 1 ? __builtin_amdgcn_update_dpp(0, b, 0x55, 0xF, 0xF, false)
              : k == 2 ? __builtin_amdgcn_update_dpp(0, b, 0xAA, 0xF, 0xF, false)
                       : __builtin_amdgcn_update_dpp(0, b, 0xFF, 0xF, 0xF, false);
  return __builtin_bit_cast(float, r);
}

// argmax_row of at most four values in registers.
__device__ __forceinline__ int argmax4(const float (&v)[4], int K) {
  int best = K == 1 && v[0] > 0.5f ? 1 : 0;
  float top = v[0];
#pragma unroll
  for (int j = 1; j < 4; ++j)
    if (j < K && v[j] > top) {   // strict: the lowest index wins ties
      top = v[j];
      best = j;
    }
  return best;
}

// LDS row stride of W1 (floats): a multiple of 4 whose quarter is odd, so the
// 16 rows x 4 columns of an operand read fall in 64 different banks.
constexpr int fwr_stride(int ns) { return (ns & 1) ? 4 * ns : 4 * ns + 4; }

// NS: 4-feature steps of the contraction, ceil(D / 4); ACT: 0 sigma, 1 tanh;
// STORE: the hidden activations are written (forward) or not (predictions).
// The registers allow four waves per SIMD without the stores up to 36 inputs, else
// three (what fits without spilling), so that one wave's products overlap the
// others' activations; the launch has four workgroups per CU up to 40 KB of LDS,
// else two (1,048,576 rows of 33-256-3, 41 KB: matrix cores busy 37 % of the
// cycles, the vector unit 55 %).
template <int NS, int ACT, bool STORE>
__global__ __launch_bounds__(256, NS <= 9 && !STORE ? 4 : 3) void k_forward_rows(int64_t n, int D, int H, int K, const float *__restrict__ X,
                                                      mlp_params p, float *__restrict__ A, float *__restrict__ Y,
                                                      PredictOut po) {
  constexpr int XS = fwr_stride(NS);
  extern __shared__ float4 fsm4[];
  float *ws = reinterpret_cast<float *>(fsm4);       // [HB][XS]
  const int HB = min(kFwrHB, (H + 15) / 16 * 16);
  float *b1 = ws + HB * XS;                          // [HB]
  float *w2 = b1 + HB;                               // [4][HB]
  // the wave index in a scalar register: row bases derived from it are uniform
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const bool once = H <= kFwrHB;                     // one block: staged before the rows
  auto stage = [&](int h0) {
    // lanes run over columns, 4 rows per wave and pass: no index division
    for (int h = tid >> 4; h < HB; h += 16) {
      const bool on = h0 + h < H;
      const float *src = p.W1 + (int64_t)(on ? h0 + h : 0) * D;
      float v[(NS * 4 + 15) / 16];
#pragma unroll
      for (int j = 0; j < (NS * 4 + 15) / 16; ++j) {
        const int c = l16 + 16 * j;
        v[j] = src[c < D ? c : 0];
      }
#pragma unroll
      for (int j = 0; j < (NS * 4 + 15) / 16; ++j) {
        const int c = l16 + 16 * j;
        if (c < 4 * NS) ws[h * XS + c] = on && c < D ? v[j] : 0.0f;
      }
    }
    for (int h = tid; h < HB; h += 256) {
      const bool on = h0 + h < H;
      b1[h] = on ? p.b1[h0 + h] : 0.0f;
#pragma unroll
      for (int k = 0; k < 4; ++k) w2[k * HB + h] = on && k < K ? p.W2[(int64_t)k * H + h0 + h] : 0.0f;
    }
  };
  float xa[2][NS];
  auto load_x = [&](int64_t r0) {
    const float *x = X + r0 * D;   // uniform base, 32-bit lane offsets
    const int last = (int)min((int64_t)31, n - 1 - r0);
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) {
      // a row past the end reads the last one (its results are dropped)
      const uint32_t ro = (uint32_t)(min(16 * rs + l16, last) * D);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int c = 4 * s + lg;
        const float v = x[ro + (uint32_t)(c < D ? c : 0)];
        xa[rs][s] = c < D ? v : 0.0f;
      }
    }
  };
  const int64_t stride = (int64_t)gridDim.x * 128;
  int64_t r0 = (int64_t)blockIdx.x * 128 + wave * 32;
  if (once) {
    stage(0);
    __syncthreads();
  }
  int hits = 0;
  // every wave runs the same number of rounds (the block staging has barriers)
  for (int64_t base = (int64_t)blockIdx.x * 128; base < n; base += stride, r0 += stride) {
    const bool live = r0 < n;
    if (live) load_x(r0);
    float zp[2][4][4];
#pragma unroll
    for (int rs = 0; rs < 2; ++rs)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) zp[rs][i][k] = 0.0f;
    float *Ab = STORE ? A + r0 * H : nullptr;   // this wave's rows (uniform base, 32-bit lane offsets)
    const int left = (int)min((int64_t)32, n - r0);
    for (int h0 = 0; h0 < H; h0 += kFwrHB) {
      if (!once) {
        __syncthreads();   // the previous block is no longer read
        stage(h0);
        __syncthreads();
      }
      if (!live) continue;
      const int nt = (min(kFwrHB, H - h0) + 15) / 16;
      for (int ht = 0; ht < nt; ++ht) {
        const int hl = ht * 16 + l16, h = h0 + hl;
        const float *wb = ws + hl * XS + lg;
        float wv[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) wv[s] = wb[4 * s];
        f32x4_l z[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          z[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[0][s], wv[s], z[0], 0, 0, 0);
          z[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[1][s], wv[s], z[1], 0, 0, 0);
        }
        const float bias = b1[hl];
        float w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = w2[k * HB + hl];
#pragma unroll
        for (int rs = 0; rs < 2; ++rs)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float slope;
            float a = hidden_act(ACT, z[rs][i] + bias, slope);
            if (h >= H) a = 0.0f;
            if (STORE) {
              float *row = Ab + (int64_t)(16 * rs + i) * H;
              if (16 * rs + 4 * lg + i < left && h < H) row[(uint32_t)(4 * lg * H + h)] = a;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) zp[rs][i][k] = fmaf(a, w[k], zp[rs][i][k]);
          }
      }
    }
    if (!live) continue;
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) {
      // the row sums end in all 16 lanes; lane 4 i + k keeps row i, output k
      float z2 = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float v = sum16(zp[rs][i][k]);
          z2 = l16 == 4 * i + k ? v : z2;
        }
      const int k = l16 & 3;
      const int64_t r = r0 + 16 * rs + 4 * lg + (l16 >> 2);
      const float y = sigmoid(z2 + p.b2[k < K ? k : 0]);
      if (k < K && r < n) Y[r * K + k] = y;
      if (po.labels) {
        const float y4[4] = {quad_bcast(y, 0), quad_bcast(y, 1), quad_bcast(y, 2), quad_bcast(y, 3)};
        if (k == 0 && r < n) {
          const int best = argmax4(y4, K);
          po.labels[r] = best;
          if (po.T) hits += best == argmax_row(po.T + r * K, K);
        }
      }
    }
  }
  if (po.labels && po.T) {
    __shared__ int part[4];
    for (int off = 32; off >= 1; off >>= 1) hits += __shfl_xor(hits, off, kWave);
    if (lane == 0) part[wave] = hits;
    __syncthreads();
    if (tid == 0) atomicAdd(po.correct, (part[0] + part[1]) + (part[2] + part[3]));
  }
}

__global__ __launch_bounds__(256) void k_step(int D, int H, int K, mlp_params p, mlp_params g,
                                              float *__restrict__ comp, float lr, float mu,
                                              float *__restrict__ vel) {
  const int64_t P = (int64_t)D * H + H + (int64_t)H * K + K;
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= P) return;
  float *w;
  const float *gr;
  const int64_t oB1 = (int64_t)D * H, oW2 = oB1 + H, oB2 = oW2 + (int64_t)H * K;
  if (q < oB1) { w = p.W1 + q; gr = g.W1 + q; }
  else if (q < oW2) { w = p.b1 + (q - oB1); gr = g.b1 + (q - oB1); }
  else if (q < oB2) { w = p.W2 + (q - oW2); gr = g.W2 + (q - oW2); }
  else { w = p.b2 + (q - oB2); gr = g.b2 + (q - oB2); }
  float wv = *w, c = comp ? comp[q] : 0.0f;
  float step = *gr;
  if (vel) {   // heavy-ball momentum: v <- mu v + g, theta <- theta - lr v
    step = fmaf(mu, vel[q], step);
    vel[q] = step;
  }
  gd_update(wv, c, lr, step, comp != nullptr);
  *w = wv;
  if (comp) comp[q] = c;
}

}  // namespace mlpk

namespace mlpk {

__global__ void k_fill_i32(int32_t *p, int32_t v) { *p = v; }

__global__ __launch_bounds__(256) void k_copy(int64_t m, const float *__restrict__ src, float *__restrict__ dst) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < m) dst[q] = src[q];
}

__global__ __launch_bounds__(256) void k_eval_batched(const mlp_batch_item *__restrict__ items, int D, int K,
                                                      const float *__restrict__ X, const float *__restrict__ T,
                                                      const float *__restrict__ theta, float *__restrict__ loss,
                                                      int32_t *__restrict__ correct) {
  const mlp_batch_item it = items[blockIdx.x];
  const int N = it.n_rows, H = it.n_hidden;
  const float *W1 = theta + it.p_off, *b1 = W1 + (int64_t)H * D, *W2 = b1 + H, *b2 = W2 + (int64_t)K * H;
  float sq = 0.0f;
  int hit = 0;
  for (int r = threadIdx.x; r < N; r += blockDim.x) {
    const float *x = X + (it.x_off + r) * D;
    const float *t = T + (it.x_off + r) * K;
    float z2[MLP_SMALL_MAX_OUT];
#pragma unroll
    for (int k = 0; k < MLP_SMALL_MAX_OUT; ++k) z2[k] = k < K ? b2[k] : 0.0f;
    for (int h = 0; h < H; ++h) {
      const float *w = W1 + (int64_t)h * D;
      float z = b1[h];
      for (int d = 0; d < D; ++d) z = fmaf(x[d], w[d], z);
      const float a = sigmoid(z);
#pragma unroll
      for (int k = 0; k < MLP_SMALL_MAX_OUT; ++k)
        if (k < K) z2[k] = fmaf(a, W2[(int64_t)k * H + h], z2[k]);
    }
    float y[MLP_SMALL_MAX_OUT];
#pragma unroll
    for (int k = 0; k < MLP_SMALL_MAX_OUT; ++k) {
      y[k] = sigmoid(z2[k]);
      if (k < K) {
        const float e = y[k] - t[k];
        sq = fmaf(e, e, sq);
      }
    }
    hit += argmax_row(y, K) == argmax_row(t, K);
  }
  __shared__ float ps[4];
  __shared__ int ph[4];
  float v = wave_sum(sq);
  int c = hit;
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, kWave);
  if ((threadIdx.x & 63) == 0) {
    ps[threadIdx.x >> 6] = v;
    ph[threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    loss[blockIdx.x] = ((ps[0] + ps[1]) + (ps[2] + ps[3])) / ((float)N * (float)K);
    if (correct) correct[blockIdx.x] = (ph[0] + ph[1]) + (ph[2] + ph[3]);
  }
}

// The same for n_in <= 64: the network's hidden tiles (16 units) are split
// over the workgroup's 4 waves and its rows taken 32 at a time, z1 on
// v_mfma_f32_16x16x4_f32 with every operand straight from global memory (each
// is used once or twice), the output sums meeting in LDS in wave order.
// A network is a few microseconds of latency, not of work, so the chip is
// filled with one network per workgroup; one thread per row left 230 of 256
// threads idle on a 25-row fold and walked W1 alone (4096 networks of up to
// 64 units: 250 us).  NS = ceil(n_in / 4).
template <int NS>
__global__ __launch_bounds__(256, 4) void k_eval_tiled(const mlp_batch_item *__restrict__ items, int D, int K,
                                                    const float *__restrict__ X, const float *__restrict__ T,
                                                    const float *__restrict__ theta, float *__restrict__ loss,
                                                    int32_t *__restrict__ correct) {
  __shared__ float zs[2][4][32][5];   // [buffer][wave][row][output], rows 5 apart: distinct banks
  __shared__ float ps[2];
  __shared__ int ph[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const mlp_batch_item it = items[blockIdx.x];
  const int N = it.n_rows, H = it.n_hidden, HT = (H + 15) / 16;
  const float *W1 = theta + it.p_off, *b1 = W1 + (int64_t)H * D, *W2 = b1 + H, *b2 = W2 + (int64_t)K * H;
  const float *Xn = X + it.x_off * D, *Tn = T + it.x_off * K;
  float total = 0.0f, sq = 0.0f;   // (the sum of a long fold in two levels)
  int hit = 0, buf = 0;
  for (int r0 = 0; r0 < N; r0 += 32, buf ^= 1) {
    const int rows = min(32, N - r0);
    // this thread's output of the round (waves 0 and 1): its target and bias
    // load with the operands, not after the barrier
    const int rt = (tid >> 2) & 31, kt = tid & 3;
    const bool on_t = rt < rows && kt < K;
    const float tl = gld(gbuf(Tn + (int64_t)r0 * K, (uint32_t)(rows * K) * 4u), kt < K ? 4u * (rt * K + kt) : kNoLoad);
    const float bl = gld(gbuf(b2, K * 4u), 4u * kt);
    float zp[2][4][4];
#pragma unroll
    for (int rs = 0; rs < 2; ++rs)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) zp[rs][i][k] = 0.0f;
    if (wave < HT) {
      float xa[2][NS];
      const __amdgpu_buffer_rsrc_t xc = gbuf(Xn + (int64_t)r0 * D, (uint32_t)(rows * D) * 4u);
      const __amdgpu_buffer_rsrc_t w1r = gbuf(W1, (uint32_t)(H * D) * 4u);
      const __amdgpu_buffer_rsrc_t b1r = gbuf(b1, (uint32_t)H * 4u), w2r = gbuf(W2, (uint32_t)(K * H) * 4u);
      uint32_t co[NS];   // column offsets of the lane, past the end for padding
#pragma unroll
      for (int s = 0; s < NS; ++s) co[s] = 4 * s + lg < D ? 4u * (4 * s + lg) : kNoLoad;
#pragma unroll
      for (int rs = 0; rs < 2; ++rs)
#pragma unroll
        for (int s = 0; s < NS; ++s)
          xa[rs][s] = gld(xc, co[s] + 4u * (uint32_t)((16 * rs + l16) * D));
      for (int t = wave; t < HT; t += 4) {
        const int h = 16 * t + l16;
        const bool hon = h < H;
        const uint32_t ho = 4u * (uint32_t)(h * D);   // (a row past H lies past the end)
        float wv[NS], w2[4];
#pragma unroll
        for (int s = 0; s < NS; ++s) wv[s] = gld(w1r, ho + co[s]);
        const float bias = gld(b1r, 4u * h);
#pragma unroll
        for (int k = 0; k < 4; ++k) w2[k] = gld(w2r, hon && k < K ? 4u * (uint32_t)(k * H + h) : kNoLoad);
        f32x4_l z[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          z[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[0][s], wv[s], z[0], 0, 0, 0);
          z[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[1][s], wv[s], z[1], 0, 0, 0);
        }
#pragma unroll
        for (int rs = 0; rs < 2; ++rs)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = hon ? sigmoid(z[rs][i] + bias) : 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) zp[rs][i][k] = fmaf(a, w2[k], zp[rs][i][k]);
          }
      }
    }
    // lane 4 i + k of a row group keeps row i, output k of the wave's share
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) {
      float z2 = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float v = sum16(zp[rs][i][k]);
          z2 = l16 == 4 * i + k ? v : z2;
        }
      zs[buf][wave][16 * rs + 4 * lg + (l16 >> 2)][l16 & 3] = z2;
    }
    __syncthreads();   // the next round writes the other buffer
    if (wave < 2) {
      const int r = rt, k = kt;
      const float z2 = (zs[buf][0][r][k] + zs[buf][1][r][k]) + (zs[buf][2][r][k] + zs[buf][3][r][k]);
      const float y = sigmoid(z2 + bl);
      const float t = on_t ? tl : 0.0f;
      const float e = on_t ? y - t : 0.0f;
      sq = fmaf(e, e, sq);
      const float y4[4] = {quad_bcast(y, 0), quad_bcast(y, 1), quad_bcast(y, 2), quad_bcast(y, 3)};
      const float t4[4] = {quad_bcast(t, 0), quad_bcast(t, 1), quad_bcast(t, 2), quad_bcast(t, 3)};
      if (k == 0 && r < rows) hit += argmax4(y4, K) == argmax4(t4, K);
      if ((r0 & 1023) == 992) {
        total += sq;
        sq = 0.0f;
      }
    }
  }
  if (wave < 2) {
    const float v = wave_sum(total + sq);
    for (int off = 32; off >= 1; off >>= 1) hit += __shfl_xor(hit, off, kWave);
    if (lane == 0) {
      ps[wave] = v;
      ph[wave] = hit;
    }
  }
  __syncthreads();
  if (tid == 0) {
    loss[blockIdx.x] = (ps[0] + ps[1]) / ((float)N * (float)K);
    if (correct) correct[blockIdx.x] = ph[0] + ph[1];
  }
}

// The same for networks of up to 16 units, one hidden tile, whose other waves
// would be idle above: each wave has 32-row sets of its own, no shares to meet.
// A lane ends with one output of one row.  1000 rows of 10 units and 4 inputs:
// 52 us above, 14 here, 24 with a thread per row; 20,000 rows 974, 233, 434; 4096
// networks of 25 rows and up to 16 units, 33 inputs 17.3 above, 9.8 here.
template <int NS>
__global__ __launch_bounds__(256) void k_eval_rows(const mlp_batch_item *__restrict__ items, int D, int K,
                                                   const float *__restrict__ X, const float *__restrict__ T,
                                                   const float *__restrict__ theta, float *__restrict__ loss,
                                                   int32_t *__restrict__ correct) {
  __shared__ float ps[4];
  __shared__ int ph[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), NW = blockDim.x >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const mlp_batch_item it = items[blockIdx.x];
  const int N = it.n_rows, H = it.n_hidden;
  const float *W1 = theta + it.p_off, *b1 = W1 + H * D, *W2 = b1 + H, *b2 = W2 + K * H;
  const float *Xn = X + it.x_off * D, *Tn = T + it.x_off * K;
  const bool hon = l16 < H;
  uint32_t co[NS];   // column offsets of the lane, past the end for padding
#pragma unroll
  for (int s = 0; s < NS; ++s) co[s] = 4 * s + lg < D ? 4u * (4 * s + lg) : kNoLoad;
  float wv[NS], w2[4];
  const __amdgpu_buffer_rsrc_t w1r = gbuf(W1, (uint32_t)(H * D) * 4u);
#pragma unroll
  for (int s = 0; s < NS; ++s) wv[s] = gld(w1r, 4u * (uint32_t)(l16 * D) + co[s]);
  const float bias = gld(gbuf(b1, (uint32_t)H * 4u), 4u * l16);
#pragma unroll
  for (int k = 0; k < 4; ++k) w2[k] = gld(gbuf(W2, (uint32_t)(K * H) * 4u), hon && k < K ? 4u * (uint32_t)(k * H + l16) : kNoLoad);
  const int k = l16 & 3;   // this lane's output
  const float b2k = gld(gbuf(b2, K * 4u), 4u * k);
  float total = 0.0f, sq = 0.0f;
  int hit = 0, round = 0;
  for (int64_t r0 = 32 * wave; r0 < N; r0 += 32 * NW) {
    const int rows = (int)min((int64_t)32, N - r0);
    const __amdgpu_buffer_rsrc_t xc = gbuf(Xn + r0 * D, (uint32_t)(rows * D) * 4u);
    const __amdgpu_buffer_rsrc_t tr = gbuf(Tn + r0 * K, (uint32_t)(rows * K) * 4u);
    float xa[2][NS], tl[2];
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) {
      tl[rs] = gld(tr, k < K ? 4u * (uint32_t)((16 * rs + 4 * lg + (l16 >> 2)) * K + k) : kNoLoad);
#pragma unroll
      for (int s = 0; s < NS; ++s) xa[rs][s] = gld(xc, co[s] + 4u * (uint32_t)((16 * rs + l16) * D));
    }
    f32x4_l z[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      z[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[0][s], wv[s], z[0], 0, 0, 0);
      z[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[1][s], wv[s], z[1], 0, 0, 0);
    }
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) {
      // lane 4 i + k of a row group keeps row i, output k
      float z2 = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a = hon ? sigmoid(z[rs][i] + bias) : 0.0f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const float v = sum16(a * w2[kk]);
          z2 = l16 == 4 * i + kk ? v : z2;
        }
      }
      const int r = 16 * rs + 4 * lg + (l16 >> 2);
      const bool on = r < rows && k < K;
      const float y = sigmoid(z2 + b2k), t = on ? tl[rs] : 0.0f, e = on ? y - t : 0.0f;
      sq = fmaf(e, e, sq);
      const float y4[4] = {quad_bcast(y, 0), quad_bcast(y, 1), quad_bcast(y, 2), quad_bcast(y, 3)};
      const float t4[4] = {quad_bcast(t, 0), quad_bcast(t, 1), quad_bcast(t, 2), quad_bcast(t, 3)};
      if (k == 0 && r < rows) hit += argmax4(y4, K) == argmax4(t4, K);
    }
    if ((++round & 31) == 0) {   // (a long fold's sum in two levels)
      total += sq;
      sq = 0.0f;
    }
  }
  total = wave_sum(total + sq);
  for (int off = 32; off >= 1; off >>= 1) hit += __shfl_xor(hit, off, kWave);
  if (lane == 0) {
    ps[wave] = total;
    ph[wave] = hit;
  }
  __syncthreads();
  if (tid == 0) {
    float v = ps[0];
    int c = ph[0];
    for (int w = 1; w < NW; ++w) {
      v += ps[w];
      c += ph[w];
    }
    loss[blockIdx.x] = v / ((float)N * (float)K);
    if (correct) correct[blockIdx.x] = c;
  }
}

__global__ __launch_bounds__(256) void k_argmax(int64_t n, int K, const float *__restrict__ Y,
                                                const float *__restrict__ T, int32_t *__restrict__ labels,
                                                int32_t *__restrict__ correct) {
  int hit = 0;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const int c = argmax_row(Y + r * K, K);
    labels[r] = c;
    if (T) hit += c == argmax_row(T + r * K, K);
  }
  if (T) {
    __shared__ int part[4];
    int v = hit;
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(correct, (part[0] + part[1]) + (part[2] + part[3]));
  }
}

}  // namespace mlpk

namespace mlph {

static dim3 grid_for(int64_t n, int b) { return dim3((unsigned)((n + b - 1) / b)); }

// k_forward_rows for every contraction length and activation.
template <int NS, bool STORE>
static const void *forward_rows_kernel(int ns, int act) {
  if (ns == NS)
    return act ? (const void *)mlpk::k_forward_rows<NS, 1, STORE> : (const void *)mlpk::k_forward_rows<NS, 0, STORE>;
  if constexpr (NS < 16) return forward_rows_kernel<NS + 1, STORE>(ns, act);
  return nullptr;
}

static bool forward_rows_covers(int D, int K) { return D <= 64 && K <= 4; }

static hipError_t launch_forward_rows(int64_t n, int D, int H, int K, const float *X, mlp_params p, float *A,
                                      float *Y, mlpk::PredictOut po, int act, int n_cu, hipStream_t s) {
  const int ns = (D + 3) / 4;
  const int HB = std::min(mlpk::kFwrHB, (H + 15) / 16 * 16);
  const size_t lds = sizeof(float) * (size_t)HB * (mlpk::fwr_stride(ns) + 5);
  const void *kern = A ? forward_rows_kernel<1, true>(ns, act) : forward_rows_kernel<1, false>(ns, act);
  hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // resident workgroups: four per CU while their LDS allows it, else two
  const int per_cu = lds <= 40 * 1024 ? 4 : 2;
  const int64_t blocks = std::min<int64_t>((n + 127) / 128, (int64_t)n_cu * per_cu);
  void *args[] = {&n, &D, &H, &K, &X, &p, &A, &Y, &po};
  e = hipLaunchKernel(kern, dim3((unsigned)blocks), dim3(256), args, lds, s);
  return e == hipSuccess ? hipGetLastError() : e;
}

hipError_t launch_forward(int64_t n, int D, int H, int K, const float *X, mlp_params p, float *A,
                          float *Y, int act, int n_cu, hipStream_t s) {
  if (forward_rows_covers(D, K))
    return launch_forward_rows(n, D, H, K, X, p, A, Y, mlpk::PredictOut{nullptr, nullptr, nullptr}, act, n_cu, s);
  if (D <= mlpk::kFwdMaxD && K <= mlpk::kLayerMaxOut) {
    const int XS = (D + 3) / 4 * 4 + 1;
    const size_t lds = sizeof(float) * ((size_t)(mlpk::kFwdRows + mlpk::kFwdHB) * XS +
                                        mlpk::kLayerMaxOut * mlpk::kFwdHB + mlpk::kFwdHB);
    using mlpk::k_forward_tiled;
    using mlpk::kLayerMaxOut;
    const void *kern = K <= 4 ? (act ? (const void *)k_forward_tiled<4, 1> : (const void *)k_forward_tiled<4, 0>)
                              : (act ? (const void *)k_forward_tiled<kLayerMaxOut, 1>
                                     : (const void *)k_forward_tiled<kLayerMaxOut, 0>);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t blocks = (n + mlpk::kFwdRows - 1) / mlpk::kFwdRows;
    void *args[] = {&n, &D, &H, &K, &X, &p, &A, &Y};
    e = hipLaunchKernel(kern, dim3((unsigned)blocks), dim3(256), args, lds, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
  }
  hipLaunchKernelGGL(mlpk::k_forward, grid_for(n, 256), dim3(256), 0, s, n, D, H, K, X, p, A, Y, act);
  return hipGetLastError();
}

}  // namespace mlph

namespace mlpk {

// Cross-validation selection.  k_cv_means: a wave owns gpw (<= 64) groups,
// lane q group g0 + q, and scans every net 64 at a time: a ballot finds the
// nets of its groups, which it adds one by one in increasing order, so a
// mean is one fixed-order float32 sum.  k_cv_best: a (mean, group) minimum,
// ties to the lower group.  (One workgroup with a thread per group reading
// every (loss, group) pair from LDS took 299 us for 4096 nets in 820 groups.)
// k_cv_small: both in one workgroup, for few nets and groups.
constexpr int kSelU = 8;   // 64-net blocks whose loads are in flight together

// The mean of group g0 + lane (lanes below m) over all n nets, U blocks of 64 at
// a time.
template <int U>
__device__ __forceinline__ float cv_mean(const float *__restrict__ loss, const int32_t *__restrict__ group, int n,
                                         int g0, int m, int lane) {
  float sum = 0.0f;
  int cnt = 0;
  for (int64_t c0 = 0; c0 < n; c0 += 64 * U) {
    float lv[U];
    int gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = c0 + 64 * u + lane;
      lv[u] = loss[i < n ? i : 0];
      gv[u] = i < n ? group[i] : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint64_t hits = __ballot(gv[u] >= g0 && gv[u] - g0 < m);
      while (hits) {
        const int j = __builtin_ctzll(hits);
        hits &= hits - 1;
        const int q = __builtin_amdgcn_readlane(gv[u], j) - g0;
        const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lv[u]), j));
        if (lane == q) {
          sum += v;
          cnt += 1;
        }
      }
    }
  }
  const float v = cnt ? sum / (float)cnt : __builtin_inff();
  return v < __builtin_inff() ? v : __builtin_inff();   // (NaN or +inf: +inf)
}

__global__ __launch_bounds__(256) void k_cv_means(const float *__restrict__ loss, const int32_t *__restrict__ group,
                                                  int n, int ng, int gpw, float *__restrict__ mean) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if ((int64_t)w * gpw >= ng) return;   // whole waves leave
  const int g0 = w * gpw, m = min(gpw, ng - g0);
  const float v = cv_mean<kSelU>(loss, group, n, g0, m, lane);
  if (lane < m) mean[g0 + lane] = v;
}

constexpr int kSelThreads = 1024;
// The workgroup's lowest (mean, group) to best[0]; every thread brings its own.
__device__ __forceinline__ void cv_lowest(float mv, int mi, int32_t *best) {
  __shared__ float bv[kSelThreads / kWave];
  __shared__ int32_t bi[kSelThreads / kWave];
  const int t = threadIdx.x;
  for (int off = 32; off >= 1; off >>= 1) {
    const float v = __shfl_xor(mv, off, kWave);
    const int i = __shfl_xor(mi, off, kWave);
    if (v < mv || (v == mv && i < mi)) {
      mv = v;
      mi = i;
    }
  }
  if ((t & 63) == 0) {
    bv[t >> 6] = mv;
    bi[t >> 6] = mi;
  }
  __syncthreads();
  if (t != 0) return;
  for (int w = 1; w < (int)(blockDim.x / kWave); ++w)
    if (bv[w] < mv || (bv[w] == mv && bi[w] < mi)) {
      mv = bv[w];
      mi = bi[w];
    }
  best[0] = mi == 0x7fffffff ? 0 : mi;
}

__global__ __launch_bounds__(kSelThreads) void k_cv_best(const float *__restrict__ mean, int ng,
                                                         int32_t *__restrict__ best) {
  float mv = __builtin_inff();
  int mi = 0x7fffffff;
  for (int g = threadIdx.x; g < ng; g += kSelThreads) {
    const float v = mean[g];
    if (v < mv || (v == mv && g < mi)) {
      mv = v;
      mi = g;
    }
  }
  cv_lowest(mv, mi, best);
}

__global__ __launch_bounds__(kSelThreads) void k_cv_small(const float *__restrict__ loss,
                                                          const int32_t *__restrict__ group, int n, int ng, int gpw,
                                                          float *mean, int32_t *best) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  float mv = __builtin_inff();
  int mi = 0x7fffffff;
  for (int g0 = wave * gpw; g0 < ng + wave * gpw; g0 += gpw * (int)(blockDim.x >> 6)) {   // as often in every wave
    const int m = min(gpw, ng - g0), g = g0 + lane;   // (m <= 0: no group is left)
    const float v = cv_mean<2>(loss, group, n, g0, m, lane);
    if (ng <= kSelThreads) __syncthreads();   // one pass: the means may lie over what they are made of
    if (lane < m) {
      mean[g] = v;
      if (v < mv || (v == mv && g < mi)) {
        mv = v;
        mi = g;
      }
    }
  }
  cv_lowest(mv, mi, best);
}

}  // namespace mlpk

namespace mlph {

constexpr int kCvSmallNets = 128, kCvSmallGroups = 4096;
hipError_t launch_cv_select(const float *loss, const int32_t *group, int n_nets, int n_groups, float *group_mean,
                            int32_t *best, hipStream_t s) {
  // few nets: one launch instead of two (64 nets, 820 groups 4.3 us on the device
  // against 5.6, 4096 groups 5.6 / 7.1; 128 nets 4.5 / 5.8, 6.4 / 7.2; with the
  // nets of a group one after the other in one wave, 256 nets gain nothing)
  // means over losses or groups: in one workgroup, which writes them when all are formed
  const bool over = n_groups <= mlpk::kSelThreads && (overlap(group_mean, n_groups, loss, n_nets) ||
                                         overlap(group_mean, n_groups, reinterpret_cast<const float *>(group), n_nets));
  if (over || (n_nets <= kCvSmallNets && n_groups <= kCvSmallGroups)) {
    const int waves = std::min(16, n_groups), per = std::min(64, (n_groups + waves - 1) / waves);
    hipLaunchKernelGGL(mlpk::k_cv_small, dim3(1), dim3(64 * waves), 0, s, loss, group, n_nets, n_groups, per,
                       group_mean, best);
    return hipGetLastError();
  }
  // one group per wave until the waves fill the chip, then several
  const int gpw = std::min(64, (n_groups + 4095) / 4096);
  const int waves = (n_groups + gpw - 1) / gpw;
  hipLaunchKernelGGL(mlpk::k_cv_means, dim3((waves + 3) / 4), dim3(256), 0, s, loss, group, n_nets, n_groups, gpw,
                     group_mean);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mlpk::k_cv_best, dim3(1), dim3(mlpk::kSelThreads), 0, s, group_mean, n_groups, best);
  return hipGetLastError();
}

// k_eval_tiled or k_eval_rows for every contraction length.
template <int NS, bool ROWS>
static auto eval_kernel(int ns) -> decltype(&mlpk::k_eval_batched) {
  if constexpr (ROWS) {
    if (ns == NS) return mlpk::k_eval_rows<NS>;
  } else {
    if (ns == NS) return mlpk::k_eval_tiled<NS>;
  }
  if constexpr (NS < 16) return eval_kernel<NS + 1, ROWS>(ns);
  return mlpk::k_eval_batched;   // n_in > 64: one thread per row
}

// One thread per row above 64 inputs, and where there are rows for the threads and
// a row is little more than its sigmoids, of which 16-unit tiles evaluate the
// padding too.  Threads / tiles, 4096 networks of 1000 rows: 1 input, 10 units
// 62 / 110 us, 64 units 262 / 331; 3 inputs, 10 units 92 / 111; 4 inputs, 6 units
// 101 / 111, 10 units 154 / 111; of 100..128 rows, 1 input, 10 units 13 / 17.  One
// network of 1000 rows, 1 input: 6 units 11.5 / 13.9, 10 units 15.6 / 13.9.
hipError_t launch_eval_batched(const mlp_batch_item *items_dev, int n_nets, int max_rows, int max_hidden, int D, int K,
                               const float *X, const float *T, const float *theta, float *loss, int32_t *correct,
                               hipStream_t s) {
  const bool rows = max_hidden <= 16, full = n_nets >= 1024;
  const int64_t unit = (D + 4) * (int64_t)max_hidden;
  const bool threads = D > 64 || (max_rows >= (full ? 96 : 256) && unit <= (full ? 72 : 36)) ||
                       (full && max_rows >= 256 && D == 1);
  const int ns = (D + 3) / 4;
  const auto kern = threads ? mlpk::k_eval_batched : rows ? eval_kernel<1, true>(ns) : eval_kernel<1, false>(ns);
  const int waves = threads || !rows ? 4 : std::min(4, (max_rows + 31) / 32);
  hipLaunchKernelGGL(kern, dim3(n_nets), dim3(64 * waves), 0, s, items_dev, D, K, X, T, theta, loss, correct);
  return hipGetLastError();
}

hipError_t launch_predict(int64_t n, int D, int H, int K, const float *X, mlp_params p, float *Y,
                          int32_t *labels, const float *T, int32_t *correct, int act, int n_cu, hipStream_t s) {
  auto fill = [&] {
    if (T) hipLaunchKernelGGL(mlpk::k_fill_i32, dim3(1), dim3(1), 0, s, correct, 0);
    return hipGetLastError();
  };
  // one pass unless labels or count lie over what the pass reads, or over Y:
  // these are then written after it
  const float *lf = reinterpret_cast<const float *>(labels), *cf = reinterpret_cast<const float *>(correct);
  const struct { const float *p; int64_t n; } ins[] = {{X, n * D}, {Y, n * K}, {p.W1, (int64_t)D * H},
                                                       {p.b1, H}, {p.W2, (int64_t)H * K}, {p.b2, K}};
  bool one = forward_rows_covers(D, K);
  for (const auto &i : ins) one = one && !overlap(lf, n, i.p, i.n) && !(T && overlap(cf, 1, i.p, i.n));
  hipError_t e = one ? fill() : launch_forward(n, D, H, K, X, p, nullptr, Y, act, n_cu, s);
  if (e != hipSuccess) return e;
  if (one)
    return launch_forward_rows(n, D, H, K, X, p, nullptr, Y, mlpk::PredictOut{labels, T, correct}, act, n_cu, s);
  if ((e = fill()) != hipSuccess) return e;
  // at most 512 blocks (rows in a grid-stride loop): one count add per block
  const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(512, (n + 255) / 256)));
  hipLaunchKernelGGL(mlpk::k_argmax, grid, dim3(256), 0, s, n, K, Y, T, labels, correct);
  return hipGetLastError();
}

// ws: `ws_floats` floats for the row ranges' partial gradients (packed order
// [W1 | b1 | W2 | b2 | loss] each).
template <int KO>
static hipError_t backward_ko(int64_t n, int64_t ws_floats, int D, int H, int K, const float *X, const float *A,
                              const float *Y, const float *dY, const float *T, mlp_params p, mlp_params g, float *dX,
                              float *loss, float *ws, int act, hipStream_t s) {
  const float inv_nk = 1.0f / ((float)n * (float)K);
  if (dY) loss = nullptr;
  mlpk::HiddenDelta<KO> src{A, p.W2, Y, dY, T, K, act, 2.0f / ((float)n * (float)K), g.W2, g.b2, loss, inv_nk};
  const int64_t oB1 = (int64_t)D * H, oW2 = oB1 + H, oB2 = oW2 + (int64_t)H * K, P = oB2 + K;
  const mlpk::GradDst dst{{g.W1, g.b1, g.W2, g.b2, loss}, {oB1, oW2, oB2, P, P + 1}, inv_nk};
  hipError_t e = launch_grads(n, D, H, X, src, g.W1, g.b1, ws, ws_floats, P + 1, dst, s);
  if (e != hipSuccess || !dX) return e;
  return launch_grad_dx(n, D, H, p.W1, src, dX, s);
}

hipError_t launch_backward(int64_t n, int64_t ws_floats, int D, int H, int K, const float *X,
                           const float *A, const float *Y, const float *dY, const float *T,
                           mlp_params p, mlp_params g, float *dX, float *loss, float *ws, int act,
                           hipStream_t s) {
  // Gradients or the loss over Y, dY or T: every workgroup reads these while
  // others write, so a copy in the workspace takes their place (the partials
  // get the rest of it; its size is n (H + K + 1) floats up to kBackwardChunk rows).
  const int64_t m = n * K;
  const struct { const float *p; int64_t n; } outs[] = {
      {g.W1, (int64_t)D * H}, {g.b1, H}, {g.W2, (int64_t)H * K}, {g.b2, K}, {dY ? nullptr : loss, 1}};
  for (const float **in : {&Y, &dY, &T}) {
    bool hit = false;
    for (const auto &o : outs) hit = hit || overlap(o.p, o.n, *in, m);
    if (!hit || m > ws_floats || (in == &T && dY)) continue;
    hipLaunchKernelGGL(mlpk::k_copy, grid_for(m, 256), dim3(256), 0, s, m, *in, ws);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    *in = ws;
    ws += m;
    ws_floats -= m;
  }
  if (K <= 4) return backward_ko<4>(n, ws_floats, D, H, K, X, A, Y, dY, T, p, g, dX, loss, ws, act, s);
  return backward_ko<mlpk::kLayerMaxOut>(n, ws_floats, D, H, K, X, A, Y, dY, T, p, g, dX, loss, ws, act, s);
}

hipError_t launch_step(int D, int H, int K, mlp_params p, mlp_params g, float *comp, float lr, float mu,
                       float *vel, hipStream_t s) {
  const int64_t P = (int64_t)D * H + H + (int64_t)H * K + K;
  hipLaunchKernelGGL(mlpk::k_step, grid_for(P, 256), dim3(256), 0, s, D, H, K, p, g, comp, lr, mu, vel);
  return hipGetLastError();
}

}  // namespace mlph
