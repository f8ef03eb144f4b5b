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
//   k_grad_unit    the sums of few rows: a workgroup owns one unit x 64 inputs
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

// The sums of few rows: a workgroup owns one unit and 64 inputs (a lane each),
// its 8 waves take 64-row sets in turn, a lane forming delta of one row, and
// meet in LDS in pairs.  (Eight chains per wave: a sum of n rows is n / 64
// steps deep and 6 to meet, as with a wave of lanes over the rows.)  k_grad_sum's
// 64 x 64 tiles leave a small layer to one workgroup: 512 rows of 50 -> 38
// 20.0 us a call, here 4.6; mlp_backward of 512 rows of 33-16-3 25.0 us, here 6.0,
// of 10-10-1 24.2 and 5.5 (device times).
constexpr int kUnitWaves = 8;
template <class Src>
__global__ __launch_bounds__(64 * kUnitWaves) void k_grad_unit(int64_t n, int din, int dout, int ftiles,
                                                               const float *__restrict__ X, Src src,
                                                               float *__restrict__ gW, float *__restrict__ gb) {
  constexpr int KO = Src::KO, KR = KO > 0 ? KO : 1;
  // lane sums that meet over the waves: gb, and beside an output layer gW2, gb2
  // and the squared error
  constexpr int NS = KO > 0 ? 2 + 2 * KO : 1;
  __shared__ float part[kUnitWaves][64];
  __shared__ float sums[kUnitWaves][NS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int o = blockIdx.x / ftiles, ft = blockIdx.x - o * ftiles, f = ft * 64 + lane;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, sum[NS], w2[KR], sq = 0.0f;
#pragma unroll
  for (int i = 0; i < NS; ++i) sum[i] = 0.0f;
  if constexpr (KO > 0) {
#pragma unroll
    for (int k = 0; k < KO; ++k) w2[k] = k < src.K ? src.W2[(int64_t)k * dout + o] : 0.0f;
  }
  for (int64_t r0 = wave * 64; r0 < n; r0 += 64 * kUnitWaves) {
    const int rows = (int)min((int64_t)64, n - r0);
    const __amdgpu_buffer_rsrc_t xr = gbuf(X + r0 * din, (uint32_t)(rows * din) * 4u);   // rows past n read zero
    float x[64];
#pragma unroll
    for (int j = 0; j < 64; ++j) x[j] = gld(xr, f < din ? 4u * (uint32_t)(j * din + f) : kNoLoad);
    const int64_t r = r0 + min(lane, rows - 1), q = r * dout + o;
    float d;
    if constexpr (KO > 0) {
      const float a = src.A[q];
      float bp = 0.0f, sr = 0.0f;
#pragma unroll
      for (int k = 0; k < KO; ++k) {
        float d2 = k < src.K ? src.d2(r, k, sr) : 0.0f;
        bp = fmaf(d2, w2[k], bp);
        d2 = lane < rows ? d2 : 0.0f;
        sum[1 + k] = lane < rows ? fmaf(d2, a, sum[1 + k]) : sum[1 + k];
        sum[1 + KO + k] += d2;
      }
      sq += lane < rows ? sr : 0.0f;
      d = src.slope_times(a, bp);
    } else {
      d = src.slope_times(src.Y[q], src.dY[q]);
    }
    d = lane < rows ? d : 0.0f;
    sum[0] += d;
#pragma unroll
    for (int j = 0; j < 64; ++j)
      acc[j & 7] = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(d), j)), x[j], acc[j & 7]);
  }
  part[wave][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  if (ft == 0) {   // the workgroup that also sums gb and gW2 (o == 0: gb2, the loss)
    if constexpr (KO > 0) sum[NS - 1] = sq;
    const int ns = KO > 0 ? (o == 0 ? NS : 1 + KO) : NS;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      if (i < ns) {
        const float v = wave_sum(sum[i]);
        if (lane == 0) sums[wave][i] = v;
      }
    }
  }
  __syncthreads();
  if (wave != 0) return;
  auto meet = [](float (&v)[kUnitWaves]) {
#pragma unroll
    for (int st = 1; st < kUnitWaves; st *= 2)
#pragma unroll
      for (int w = 0; w < kUnitWaves; w += 2 * st) v[w] += v[w + st];
    return v[0];
  };
  float v[kUnitWaves];
#pragma unroll
  for (int w = 0; w < kUnitWaves; ++w) v[w] = part[w][lane];
  const float g = meet(v);
  if (f < din) gW[(int64_t)o * din + f] = g;
  if (ft != 0 || lane >= NS) return;
#pragma unroll
  for (int w = 0; w < kUnitWaves; ++w) v[w] = sums[w][lane];
  const float t = meet(v);
  if (lane == 0) gb[o] = t;
  if constexpr (KO > 0) {
    const int k = lane <= KO ? lane - 1 : lane - 1 - KO;
    if (lane >= 1 && lane <= KO && k < src.K) src.gW2[(int64_t)k * dout + o] = t;
    if (o == 0 && lane > KO && k < src.K) src.gb2[k] = t;
    if (o == 0 && lane == NS - 1 && src.loss) src.loss[0] = t * src.loss_scale;
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

// Whether na floats at a and nb floats at b share memory (NULL: no).
inline bool overlap(const float *a, int64_t na, const float *b, int64_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return a && b && x < y + sizeof(float) * (uintptr_t)nb && y < x + sizeof(float) * (uintptr_t)na;
}

// Row ranges of the gradient sums: enough workgroups for about two per CU,
// each range at least 128 rows (a set for every wave: of 160 rows one wave has
// two while three wait, 33 -> 16 on 2300 rows 13.9 us, on ranges of 128 10.7),
// and no more partials than the workspace holds.
inline int64_t grad_ranges(int64_t n, int64_t tiles, int64_t Q, int64_t cap) {
  constexpr int64_t least = mlpk::kGWaves * mlpk::kGSet;
  int64_t S = (512 + tiles - 1) / tiles;
  S = S < (n + least - 1) / least ? S : (n + least - 1) / least;
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
  const int64_t even = ((n + S - 1) / S + kGSet - 1) / kGSet * kGSet;
  const int64_t per = even > kGWaves * kGSet ? even : kGWaves * kGSet;
  S = (n + per - 1) / per;
  const GradOut out{S > 1 ? ws : nullptr, Q, gW, gb};
  hipLaunchKernelGGL(k_grad_sum<Src>, dim3((unsigned)(ot * ft), (unsigned)S), dim3(64 * kGWaves), 0, s, n, din, dout,
                     per, (int)ft, X, src, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || S == 1) return e;
  hipLaunchKernelGGL(k_grad_reduce, dim3((unsigned)((Q + 63) / 64)), dim3(256), 0, s, Q, (int)S, ws, dst);
  return hipGetLastError();
}

// k_grad_unit up to these rows, workgroups, and rows x workgroups: beyond, X
// read once per unit costs more than k_grad_sum's tiles and the launch that adds
// their partials.  Microseconds on the device, here against there: 50 -> 38, 1200
// rows 7.0 / 11, 2048 10.4 / 10.9, 3000 14.0 / 11.5; 64 -> 256, 1200 rows 7.8 /
// 11, 2048 14.1 / 11.2; below an output layer 33-16-3, 512 rows 6.0 / 12.7, 2048
// 13.7 / 13.4, 2500 16.3 / 13.7; 33-1024-3, 60 rows 11.3 / 10.3, 300 16.4 / 12.7;
// with more than four outputs 64-64-16, 800 rows 19.0 / 21.6, 1200 25.1 / 21.9;
// 64-512-12, 300 rows 16 / 20, 800 27 / 21.
constexpr int64_t kUnitRows = 2048, kUnitRowsWide = 1024, kUnitGroups = 512, kUnitWork = 400000;

// The sums by the form that suits the sizes.
template <class Src>
hipError_t launch_grads(int64_t n, int din, int dout, const float *X, const Src &src, float *gW, float *gb, float *ws,
                        int64_t cap, int64_t Q, const mlpk::GradDst &dst, hipStream_t s) {
  const int64_t ft = ((int64_t)din + 63) / 64, groups = dout * ft;
  if (n > (Src::KO > 4 ? kUnitRowsWide : kUnitRows) || groups > kUnitGroups || n * groups > kUnitWork)
    return launch_grad_sum(n, din, dout, X, src, gW, gb, ws, cap, Q, dst, s);
  hipLaunchKernelGGL(mlpk::k_grad_unit<Src>, dim3((unsigned)groups), dim3(64 * mlpk::kUnitWaves), 0, s, n, din, dout,
                     (int)ft, X, src, gW, gb);
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
