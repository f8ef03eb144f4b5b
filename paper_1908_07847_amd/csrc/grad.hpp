// Gradients of a layer from its deltas, for the layer kernels (one hidden
// layer, mlp_backward) and the dense kernels (mlp_dense_backward).
//
//   gW[o][i] = sum_r delta[r][o] X[r][i],  gb[o] = sum_r delta[r][o]
//   dX[r][i] = sum_o delta[r][o] W[o][i]
//
// A source object forms delta[r][o] on the fly from what the caller holds
// (the outputs and the upstream gradient), so no delta array is written.
//
//   k_grad_sum     a workgroup owns 64 units x 64 inputs and a range of rows;
//                  its 4 waves take 32-row sets of the range in turn.  delta
//                  and X go from global memory straight into the operands of
//                  v_mfma_f32_16x16x4_f32 (M = units, N = inputs, K = rows:
//                  a lane's operand is one element, 16 lanes read 64
//                  contiguous bytes), 16 rows' loads issued together; the
//                  waves meet in LDS in a fixed order.
//   k_grad_reduce  adds the row ranges' partials of every parameter in a fixed
//                  order (not launched when one range covers all rows)
//   k_grad_dx      64 rows x 64 inputs per workgroup, delta and W staged in
//                  LDS in chunks of 64 units
//
// Bound: the gradient sums read X once per 64 units and the outputs once
// per 64 inputs; the float32 matrix-core rate bounds the products.  One wave
// per parameter walking two columns of X and delta, which this replaces,
// read a cache line per element: 50,000 rows of a 33-256-3 network took
// 3.2 ms in the sums (mlp_backward in all 3.7 ms).
#pragma once
#include "mlp_device.hpp"

namespace mlpk {

typedef float f32x4_g __attribute__((ext_vector_type(4)));

constexpr int kGT = 64;    // units and inputs per tile
constexpr int kGSet = 32;  // rows of a wave's set
constexpr int kGWaves = 4;
// Depth of the float32 sums.  A chain of matrix-core products errs like one
// rounding per row, so a wave starts every 16 rows from zero and adds the
// result to its totals, and a range adds the totals of every kGFold rows in
// memory: n rows of one range are 16 + min(n, kGFold) / 64 + n / kGFold steps
// deep, however few ranges the tiles and the workspace leave.  One chain per
// range is n / 4 deep: 262,144 rows of 33-64-3 in one range, equal terms, gW1
// off by 7.6e-4 of itself, so 3.1e-6; 512 rows of random terms 2.7e-7 and
// 1.3e-7; 40,000 rows of 1024 -> 2048 3.1e-6 and 3.5e-7.  It costs 6 % where the
// products bound (30,000 rows of 33-256-3 27.3 -> 28.9 us).
constexpr int kGFold = 16384;

// Where a parameter's gradient goes: packed [W | b | extra] order as partial
// s of `part` (stride Q), or the final arrays when one range covers all rows.
struct GradOut {
  float *part;   // [S][Q], or null: write the final arrays
  int64_t Q;
  float *gW, *gb;
};

// delta of a dense layer: dY . act'(Y), or (GIVEN) the delta itself in both
// arrays, for calls whose outputs lie over Y or dY.
template <bool GIVEN>
struct DenseDelta {
  static constexpr int KO = 0;   // no output layer above: nothing beside gW, gb
  const float *Y, *dY;
  int act;
  __device__ __forceinline__ float slope_times(float y, float s) const {
    if (GIVEN) return s;
    return act == 1 ? s * (1.0f - y * y) : s * (y * (1.0f - y));
  }
};

// delta of the hidden layer of a one-hidden-layer network: the output deltas
// d2 = dY . Y (1 - Y) (dY given, or 2 (Y - T) / (n K)) through the pre-update
// W2, times act'(A).  KO: outputs the loops run over (K <= KO).
template <int KO_>
struct HiddenDelta {
  static constexpr int KO = KO_;
  const float *A, *W2;
  const float *Y, *dY, *T;   // [n][K]; dY or T
  int K, act;
  float mse_scale;           // 2 / (n K)
  float *gW2, *gb2, *loss;   // final arrays (loss may be null)
  float loss_scale;          // 1 / (n K)
  __device__ __forceinline__ float slope_times(float a, float s) const {
    return act == 1 ? s * (1.0f - a * a) : s * a * (1.0f - a);
  }
  // output delta of row r, output k; adds the squared error to sq
  __device__ __forceinline__ float d2(int64_t r, int k, float &sq) const {
    const float y = Y[r * K + k];
    float g;
    if (dY) {
      g = dY[r * K + k];
    } else {
      const float err = y - T[r * K + k];
      sq = fmaf(err, err, sq);
      g = mse_scale * err;
    }
    return g * y * (1.0f - y);
  }
};

template <class Src>   // (two workgroups per CU, as grad_ranges counts, where no register spills for it)
__global__ __launch_bounds__(64 * kGWaves, Src::KO > 4 ? 1 : 2) void k_grad_sum(int64_t n, int din, int dout, int64_t per, int ftiles,
                                                           const float *__restrict__ X, Src src, GradOut out) {
  constexpr int KO = Src::KO, KR = KO > 0 ? KO : 1;
  __shared__ float buf[2][kGT][kGT + 1];
  __shared__ float small[kGWaves][kGT][KR + 1];   // gb and gW2 of each wave
  __shared__ float d2s[kGWaves][kGSet][KR];
  __shared__ float tail[kGWaves][KR + 1];         // gb2 and the squared error of each wave
  // the wave index in a scalar register: row bases are uniform, lanes add
  // 32-bit offsets
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int o0 = (blockIdx.x / ftiles) * kGT, f0 = (blockIdx.x % ftiles) * kGT;
  const bool first_f = f0 == 0;            // this tile also sums gb (and gW2)
  const bool first = first_f && o0 == 0;   // ... and gb2, the loss
  const int64_t r_begin = (int64_t)blockIdx.y * per, r_end = min(n, r_begin + per);

  // columns of this lane, clamped into the arrays (masked where they enter)
  int oc[4], fc[4];
  bool oo[4], fo[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    oo[t] = o0 + 16 * t + l16 < dout;
    oc[t] = oo[t] ? o0 + 16 * t + l16 : 0;
    fo[t] = f0 + 16 * t + l16 < din;
    fc[t] = fo[t] ? f0 + 16 * t + l16 : 0;
  }
  float w2[4][KR];
  if constexpr (KO > 0) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int k = 0; k < KO; ++k) w2[t][k] = k < src.K ? src.W2[(int64_t)k * dout + oc[t]] : 0.0f;
  }
  for (int64_t fold = r_begin; fold < r_end; fold += kGFold) {
    const int64_t f_end = min(r_end, fold + kGFold);
    if (fold > r_begin) __syncthreads();   // the previous fold's LDS is no longer read
    f32x4_g acc[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[t][u] = f32x4_g{0.f, 0.f, 0.f, 0.f};
    float gb[4] = {0.f, 0.f, 0.f, 0.f}, gw2[4][KR], gb2[KR], sq = 0.0f;
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      gb2[k] = 0.0f;
#pragma unroll
      for (int t = 0; t < 4; ++t) gw2[t][k] = 0.0f;
    }

    for (int64_t base = fold + wave * kGSet; base < f_end; base += kGWaves * kGSet) {
      const int rows = (int)min((int64_t)kGSet, f_end - base);
      const float *xb = X + base * din;
      if constexpr (KO > 0) {
        // output deltas of the set's rows: lane = row (the upper half idles)
        if (lane < kGSet) {
#pragma unroll
          for (int k = 0; k < KO; ++k) {
            float d = 0.0f;
            if (lane < rows && k < src.K) d = src.d2(base + lane, k, sq);
            gb2[k] += d;
            d2s[wave][lane][k] = d;
          }
        }
      }
      for (int h = 0; h < kGSet; h += 16) {   // 16 rows: their loads are issued together
        if (h >= rows) break;
        float xv[4][4], ov[4][4], uv[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int row = h + 4 * s + lg, rc = row < rows ? row : 0;
          const uint32_t xo = (uint32_t)(rc * din), oo_ = (uint32_t)(rc * dout);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            xv[s][t] = xb[xo + (uint32_t)fc[t]];
            if constexpr (KO > 0) {
              ov[s][t] = (src.A + base * dout)[oo_ + (uint32_t)oc[t]];
            } else {
              ov[s][t] = (src.Y + base * dout)[oo_ + (uint32_t)oc[t]];
              uv[s][t] = (src.dY + base * dout)[oo_ + (uint32_t)oc[t]];
            }
          }
        }
        float xm[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int u = 0; u < 4; ++u) xm[s][u] = h + 4 * s + lg < rows && fo[u] ? xv[s][u] : 0.0f;
        float dk[4][KR];
        if constexpr (KO > 0) {
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int k = 0; k < KO; ++k) dk[s][k] = d2s[wave][h + 4 * s + lg][k];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {   // the 16 rows from zero, then onto the totals
          f32x4_g part[4];
          float gbh = 0.0f, gw2h[KR];
#pragma unroll
          for (int k = 0; k < KR; ++k) gw2h[k] = 0.0f;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int row = h + 4 * s + lg;
            const bool on = row < rows && oo[t];
            float d;
            if constexpr (KO > 0) {
              const float a = on ? ov[s][t] : 0.0f;
              float bp = 0.0f;
#pragma unroll
              for (int k = 0; k < KO; ++k) {
                bp = fmaf(dk[s][k], w2[t][k], bp);
                gw2h[k] = fmaf(dk[s][k], a, gw2h[k]);
              }
              d = src.slope_times(a, bp);
            } else {
              d = src.slope_times(ov[s][t], uv[s][t]);
            }
            d = on ? d : 0.0f;
            gbh += d;
#pragma unroll
            for (int u = 0; u < 4; ++u)
              part[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(d, xm[s][u], s ? part[u] : f32x4_g{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          }
          gb[t] += gbh;
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[t][u] += part[u];
          if constexpr (KO > 0) {
#pragma unroll
            for (int k = 0; k < KO; ++k) gw2[t][k] += gw2h[k];
          }
        }
      }
    }

    // ---- the four waves meet in a fixed order: (w0 + w2) + (w1 + w3), and add
    // what this thread wrote for the range's earlier folds.  Lane
    // (input l16, group lg) holds units 4 lg .. 4 lg + 3 of each 16 x 16 tile.
    auto put = [&](int b, bool add) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float *p = &buf[b][16 * t + 4 * lg + i][16 * u + l16];
            *p = add ? acc[t][u][i] + *p : acc[t][u][i];
          }
    };
    if (wave >= 2) put(wave - 2, false);
    if (first_f) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float v = sum_rows(gb[t]);
        if (lg == 0) small[wave][16 * t + l16][0] = v;
        if constexpr (KO > 0) {
#pragma unroll
          for (int k = 0; k < KO; ++k) {
            const float g = sum_rows(gw2[t][k]);
            if (lg == 0) small[wave][16 * t + l16][1 + k] = g;
          }
        }
      }
      if constexpr (KO > 0) {
        if (first) {
#pragma unroll
          for (int k = 0; k < KO; ++k) {
            const float v = wave_sum(gb2[k]);
            if (lane == 0) tail[wave][k] = v;
          }
          sq = wave_sum(sq);
          if (lane == 0) tail[wave][KO] = sq;
        }
      }
    }
    __syncthreads();
    if (wave < 2) put(wave, true);
    __syncthreads();
    auto store = [&](float *p, float v) { *p = fold == r_begin ? v : *p + v; };
    float *pw = out.part ? out.part + (int64_t)blockIdx.y * out.Q : nullptr;
    float *gW = pw ? pw : out.gW;
    for (int q = tid; q < kGT * kGT; q += 64 * kGWaves) {
      const int o = q / kGT, f = q % kGT;
      if (o0 + o < dout && f0 + f < din) store(gW + (int64_t)(o0 + o) * din + f0 + f, buf[0][o][f] + buf[1][o][f]);
    }
    if (first_f) {
      auto waves4 = [&](int o, int c) { return (small[0][o][c] + small[2][o][c]) + (small[1][o][c] + small[3][o][c]); };
      const int64_t oB = (int64_t)dout * din;
      if (tid < kGT && o0 + tid < dout) store((pw ? pw + oB : out.gb) + o0 + tid, waves4(tid, 0));
      if constexpr (KO > 0) {
        float *g2 = pw ? pw + oB + dout : src.gW2;
        for (int q = tid; q < kGT * src.K; q += 64 * kGWaves) {
          const int k = q / kGT, o = q % kGT;
          if (o0 + o < dout) store(g2 + (int64_t)k * dout + o0 + o, waves4(o, 1 + k));
        }
        if (first && tid <= KO) {
          const float v = (tail[0][tid] + tail[2][tid]) + (tail[1][tid] + tail[3][tid]);
          const int64_t oT = oB + dout + (int64_t)src.K * dout;
          if (tid < src.K) store((pw ? pw + oT : src.gb2) + tid, v);
          if (tid == KO) {
            if (pw) store(pw + oT + src.K, v);
            else if (src.loss) store(src.loss, v * src.loss_scale);
          }
        }
      }
    }
  }
}

// Final arrays of a reduction: packed offsets [0, e0) go to p0, [e0, e1) to
// p1, and so on; the last entry (the loss) is scaled and may be dropped.
struct GradDst {
  float *p[5];
  int64_t end[5];
  float scale;   // of the last entry
};

// 64 parameters per workgroup; the 4 waves each add a quarter of the partials
// (8 loads in flight per lane) and meet in a fixed order.
static __global__ __launch_bounds__(256) void k_grad_reduce(int64_t Q, int S, const float *__restrict__ part, GradDst dst) {
  __shared__ float sm[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t q = (int64_t)blockIdx.x * 64 + lane, qc = q < Q ? q : 0;
  const int s0 = S * wave / 4, s1 = S * (wave + 1) / 4;
  float sum = 0.0f;
  int s = s0;
  for (; s + 8 <= s1; s += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(s + u) * Q + qc];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += v[u];
  }
  for (; s < s1; ++s) sum += part[(int64_t)s * Q + qc];
  sm[wave][lane] = sum;
  __syncthreads();
  if (wave != 0 || q >= Q) return;
  const float v = (sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]);
  int64_t b = 0;
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    if (q >= b && q < dst.end[j]) {
      if (dst.p[j]) dst.p[j][q - b] = j == 4 ? v * dst.scale : v;
      return;
    }
    b = dst.end[j];
  }
}

template <class Src>
__global__ __launch_bounds__(256) void k_grad_dx(int64_t n, int din, int dout, const float *__restrict__ W, Src src,
                                                 float *__restrict__ dX) {
  constexpr int KO = Src::KO, KR = KO > 0 ? KO : 1;
  __shared__ float ds[kGT][kGT + 1];   // [row][unit]
  __shared__ float ws[kGT][kGT + 2];   // [unit][input]
  __shared__ float d2s[kGT][KR];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lg = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kGT;
  const int f0 = blockIdx.y * kGT, rows = (int)min((int64_t)kGT, n - r0);
  if constexpr (KO > 0) {
    float sq = 0.0f;
    for (int q = tid; q < kGT * KO; q += 256) {
      const int r = q / KO, k = q % KO;
      d2s[r][k] = r < rows && k < src.K ? src.d2(r0 + r, k, sq) : 0.0f;
    }
  }
  f32x4_g acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f32x4_g{0.f, 0.f, 0.f, 0.f};
  for (int o0 = 0; o0 < dout; o0 += kGT) {
    __syncthreads();   // the previous chunk is no longer read (and d2s is written)
    const int o = o0 + lane;
    const bool on = o < dout;
    float w2[KR];
    if constexpr (KO > 0) {
#pragma unroll
      for (int k = 0; k < KO; ++k) w2[k] = k < src.K && on ? src.W2[(int64_t)k * dout + o] : 0.0f;
    }
    // lanes run over units: 16 rows per wave
    float yv[16], uv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int r = wave * 16 + j;
      const int64_t at = (r0 + (r < rows ? r : 0)) * dout + (on ? o : 0);
      if constexpr (KO > 0) {
        yv[j] = src.A[at];
      } else {
        yv[j] = src.Y[at];
        uv[j] = src.dY[at];
      }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int r = wave * 16 + j;
      float s;
      if constexpr (KO > 0) {
        s = 0.0f;
#pragma unroll
        for (int k = 0; k < KO; ++k) s = fmaf(d2s[r][k], w2[k], s);
      } else {
        s = uv[j];
      }
      ds[r][lane] = r < rows && on ? src.slope_times(yv[j], s) : 0.0f;
    }
    // W chunk: lanes run over inputs
    {
      const int f = f0 + lane;
      const bool fon = f < din;
      float wv[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int u = o0 + wave * 16 + j;
        wv[j] = W[(int64_t)(u < dout ? u : 0) * din + (fon ? f : 0)];
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) ws[wave * 16 + j][lane] = fon && o0 + wave * 16 + j < dout ? wv[j] : 0.0f;
    }
    __syncthreads();
    const int ksteps = (min(kGT, dout - o0) + 3) / 4;
    for (int s = 0; s < ksteps; ++s) {
      const float a = ds[wave * 16 + l16][4 * s + lg];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ws[4 * s + lg][16 * t + l16], acc[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int f = f0 + 16 * t + l16;
    if (f >= din) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = wave * 16 + 4 * lg + i;
      if (r < rows) dX[(r0 + r) * din + f] = acc[t][i];
    }
  }
}

}  // namespace mlpk

namespace mlph {

// Row ranges of the gradient sums: enough workgroups for about two per CU,
// each range at least 128 rows (a set for every wave), and no more partials
// than the workspace holds.  Up to 512 rows one range is used, for one launch
// less (15.4 us at 300 rows, 20.0 at 512; with ranges 13.6 at 513 and a launch
// more, which callers at these sizes are bound by).
inline int64_t grad_ranges(int64_t n, int64_t tiles, int64_t Q, int64_t cap) {
  if (n <= 512) return 1;
  int64_t S = (512 + tiles - 1) / tiles;
  S = S < n / 128 ? S : n / 128;
  S = S < cap / Q ? S : cap / Q;
  S = S < 65535 ? S : 65535;
  return S < 1 ? 1 : S;
}

// Launches the sums (and their reduction).  ws holds `cap` floats; dst lists
// the final arrays of the packed order, Q their total length.
template <class Src>
hipError_t launch_grad_sum(int64_t n, int din, int dout, const float *X, const Src &src, float *gW, float *gb,
                           float *ws, int64_t cap, int64_t Q, const mlpk::GradDst &dst, hipStream_t s) {
  using namespace mlpk;
  const int64_t ot = (dout + kGT - 1) / kGT, ft = (din + kGT - 1) / kGT;
  int64_t S = grad_ranges(n, ot * ft, Q, cap);
  const int64_t per = ((n + S - 1) / S + kGSet - 1) / kGSet * kGSet;
  S = (n + per - 1) / per;
  const GradOut out{S > 1 ? ws : nullptr, Q, gW, gb};
  hipLaunchKernelGGL(k_grad_sum<Src>, dim3((unsigned)(ot * ft), (unsigned)S), dim3(64 * kGWaves), 0, s, n, din, dout,
                     per, (int)ft, X, src, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || S == 1) return e;
  hipLaunchKernelGGL(k_grad_reduce, dim3((unsigned)((Q + 63) / 64)), dim3(256), 0, s, Q, (int)S, ws, dst);
  return hipGetLastError();
}

template <class Src>
hipError_t launch_grad_dx(int64_t n, int din, int dout, const float *W, const Src &src, float *dX, hipStream_t s) {
  using namespace mlpk;
  hipLaunchKernelGGL(k_grad_dx<Src>, dim3((unsigned)((n + kGT - 1) / kGT), (unsigned)((din + kGT - 1) / kGT)),
                     dim3(256), 0, s, n, din, dout, W, src, dX);
  return hipGetLastError();
}

}  // namespace mlph
