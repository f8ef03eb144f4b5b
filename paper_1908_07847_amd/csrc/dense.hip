// One fully connected layer and its adjoint: the building block of networks
// with several hidden layers (section 2.2's layer, stacked; the paper's
// network has one hidden layer).
//
//   k_dense_fwd<ACT>  Y = act(X W^T + b); a workgroup computes 64 rows x 64
//                     outputs, 16 rows per wave, on v_mfma_f32_16x16x4_f32
//                     with X and W staged in LDS in chunks of 64 inputs
//   adjoint           grad.hpp: dZ = dY . act'(Y) (act' from the layer's
//                     output) is formed where the gradient sums gW = dZ^T X,
//                     gb = sum dZ and the optional dX = dZ W consume it; row
//                     sums run in a fixed order (bitwise repeatable)
//   k_dense_dz        dZ into the workspace first, where an output lies over Y or dY
//   k_update          theta <- theta - lr g over a packed parameter vector,
//                     optionally Kahan-compensated
//   k_mse_grad        the error of section 2.2 read as the mean squared error,
//                     L = sum (Y-T)^2 / (n K), and dL/dY = 2 (Y-T) / (n K); one
//                     workgroup, threads strided over the entries, a fixed-order
//                     block sum (bitwise repeatable)
// ACT: 0 the sigmoid of Equation 1, 1 tanh.
#include "grad.hpp"
#include "mlp_device.hpp"

namespace mlpk {

constexpr int kDR = 64, kDO = 64, kDK = 64;

typedef float f32x4_d __attribute__((ext_vector_type(4)));

template <int ACT>
__device__ __forceinline__ float dense_act(float z) {
  float slope;
  return hidden_act(ACT, z, slope);
}

// Staging: lanes run over a chunk's 64 inputs, each wave over 16 of the 64
// rows (and outputs), so addresses need no division and all 32 loads of a
// thread are in flight together; the operand rows are 4 past a multiple of 64
// floats apart.  20,000 rows of 64 -> 256 (tanh): 48 us with chunks of 32
// indexed element by element, 27 us with this.
template <int ACT>
__global__ __launch_bounds__(256) void k_dense_fwd(int64_t n, int din, int dout, const float *__restrict__ X,
                                                   const float *__restrict__ W, const float *__restrict__ b,
                                                   float *__restrict__ Y) {
  __shared__ float xs[kDR][kDK + 4];
  __shared__ float ws[kDO][kDK + 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kDR;
  const int o0 = blockIdx.y * kDO;
  const int rows = (int)min((int64_t)kDR, n - r0), outs = min(kDO, dout - o0);
  f32x4_d acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f32x4_d{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < din; k0 += kDK) {
    // rows (outputs) past the end and inputs past din read zero
    const __amdgpu_buffer_rsrc_t xr = gbuf(X + r0 * din, (uint32_t)(rows * din) * 4u);
    const __amdgpu_buffer_rsrc_t wr = gbuf(W + (int64_t)o0 * din, (uint32_t)(outs * din) * 4u);
    const uint32_t c = k0 + lane < din ? 4u * (uint32_t)(wave * 16 * din + k0 + lane) : kNoLoad;
    float xv[16], wv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      xv[j] = gld(xr, c + 4u * (uint32_t)(j * din));
      wv[j] = gld(wr, c + 4u * (uint32_t)(j * din));
    }
    __syncthreads();   // the previous chunk is no longer read
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      xs[wave * 16 + j][lane] = xv[j];
      ws[wave * 16 + j][lane] = wv[j];
    }
    __syncthreads();
    const int ks = min(kDK, din - k0);
    const float *xa = &xs[wave * 16 + l16][lg], *wb = &ws[l16][lg];
    for (int k1 = 0; k1 < ks; k1 += 16) {   // 16 inputs: whole groups (the padding is zero)
      float a[4], w[4][4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        a[s] = xa[k1 + 4 * s];                        // A: rows x inputs
#pragma unroll
        for (int t = 0; t < 4; ++t) w[s][t] = wb[t * 16 * (kDK + 4) + k1 + 4 * s];   // B: inputs x outputs
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], w[s][t], acc[t], 0, 0, 0);
    }
  }
  // lane (output l16 of tile t, group lg) holds rows 4 lg .. 4 lg + 3 of the wave's 16
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int o = o0 + t * 16 + l16;
    if (o >= dout) continue;
    const float bo = b[o];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = r0 + wave * 16 + 4 * lg + i;
      if (r < n) Y[r * dout + o] = dense_act<ACT>(acc[t][i] + bo);
    }
  }
}

// dZ = dY . act'(Y), entry by entry, so dZ may be Y's or dY's own memory.
__global__ __launch_bounds__(256) void k_dense_dz(int64_t m, DenseDelta<false> src, float *dZ) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < m) dZ[q] = src.slope_times(src.Y[q], src.dY[q]);
}

__global__ __launch_bounds__(256) void k_update(int64_t P, float *__restrict__ theta, const float *__restrict__ g,
                                                float *__restrict__ comp, float lr) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= P) return;
  float w = theta[q], c = comp ? comp[q] : 0.0f;
  gd_update(w, c, lr, g[q], comp != nullptr);
  theta[q] = w;
  if (comp) comp[q] = c;
}

__global__ __launch_bounds__(1024) void k_mse_grad(int64_t m, float scale, const float *__restrict__ Y,
                                                   const float *__restrict__ T, float *__restrict__ dY,
                                                   float *__restrict__ loss) {
  __shared__ float part[16];
  float s = 0.0f;
  // eight entries per thread at a time, their loads in flight together
  for (int64_t q0 = threadIdx.x; q0 < m; q0 += 8 * blockDim.x) {
    float yv[8], tv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t q = q0 + (int64_t)u * blockDim.x;
      yv[u] = Y[q < m ? q : 0];
      tv[u] = T[q < m ? q : 0];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t q = q0 + (int64_t)u * blockDim.x;
      if (q < m) {
        const float e = yv[u] - tv[u];
        s = fmaf(e, e, s);
        dY[q] = 2.0f * e * scale;
      }
    }
  }
  s = wave_sum(s);
  if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) t += part[w];
    if (loss) loss[0] = t * scale;
  }
}

}  // namespace mlpk

namespace mlph {

static dim3 blocks_for(int64_t n, int per) { return dim3((unsigned)((n + per - 1) / per)); }

hipError_t launch_dense_forward(int64_t n, int din, int dout, const float *X, const float *W, const float *b,
                                int act, float *Y, hipStream_t s) {
  const dim3 grid((unsigned)((n + mlpk::kDR - 1) / mlpk::kDR), (unsigned)((dout + mlpk::kDO - 1) / mlpk::kDO));
  if (act == 1)
    hipLaunchKernelGGL(mlpk::k_dense_fwd<1>, grid, dim3(256), 0, s, n, din, dout, X, W, b, Y);
  else
    hipLaunchKernelGGL(mlpk::k_dense_fwd<0>, grid, dim3(256), 0, s, n, din, dout, X, W, b, Y);
  return hipGetLastError();
}

// ws: n dout floats, for the row ranges' partial gradients ([gW | gb] each).
template <bool GIVEN>
static hipError_t dense_backward(int64_t n, int din, int dout, const float *X, const mlpk::DenseDelta<GIVEN> &src,
                                 const float *W, float *gW, float *gb, float *dX, float *ws, int64_t ws_floats,
                                 hipStream_t s) {
  const int64_t nW = (int64_t)dout * din, Q = nW + dout;
  const mlpk::GradDst dst{{gW, gb, nullptr, nullptr, nullptr}, {nW, Q, Q, Q, Q}, 1.0f};
  const hipError_t e = launch_grads(n, din, dout, X, src, gW, gb, ws, ws_floats, Q, dst, s);
  if (e != hipSuccess || !dX) return e;
  return launch_grad_dx(n, din, dout, W, src, dX, s);
}

// An output (or the workspace) over Y or dY: the kernels read both to the end,
// in every workgroup, so dZ goes to the workspace first and they read that
// (the partial gradients then have no room: one range of rows).
hipError_t launch_dense_backward(int64_t n, int din, int dout, const float *X, const float *Y, const float *dY,
                                 const float *W, int act, float *gW, float *gb, float *dX, float *ws,
                                 hipStream_t s) {
  const int64_t m = n * dout;
  const mlpk::DenseDelta<false> src{Y, dY, act};
  const struct { const float *p; int64_t n; } outs[] = {{dX, n * din}, {gW, (int64_t)dout * din}, {gb, dout}, {ws, m}};
  for (const auto &o : outs)
    if (overlap(o.p, o.n, Y, m) || overlap(o.p, o.n, dY, m)) {
      hipLaunchKernelGGL(mlpk::k_dense_dz, blocks_for(m, 256), dim3(256), 0, s, m, src, ws);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      return dense_backward(n, din, dout, X, mlpk::DenseDelta<true>{ws, ws, act}, W, gW, gb, dX, ws, 0, s);
    }
  return dense_backward(n, din, dout, X, src, W, gW, gb, dX, ws, m, s);
}

hipError_t launch_mse_grad(int64_t n, int k, const float *Y, const float *T, float *dY, float *loss, hipStream_t s) {
  const int64_t m = n * k;
  hipLaunchKernelGGL(mlpk::k_mse_grad, dim3(1), dim3(1024), 0, s, m, 1.0f / ((float)n * (float)k), Y, T, dY, loss);
  return hipGetLastError();
}

hipError_t launch_update(int64_t P, float *theta, const float *g, float *comp, float lr, hipStream_t s) {
  hipLaunchKernelGGL(mlpk::k_update, blocks_for(P, 256), dim3(256), 0, s, P, theta, g, comp, lr);
  return hipGetLastError();
}

}  // namespace mlph
