// Small-network trainer: one workgroup trains one network, full batch, for
// all epochs in a single launch (arxiv 1908.07847, section 2.2: feed
// forward, error, backpropagation, gradient-descent update, repeated for a
// number of epochs).
//
// The net lives in LDS for the whole run: its rows X with a constant-1
// column (so b1 is the last column of W1), the targets, W1|b1, W2 and b2.
// HBM is read once at the start and written once at the end.  Each of the
// NW waves owns every NW-th 16-row tile of the batch and, per epoch:
//
//   z1^T = [W1 b1] [X 1]^T     v_mfma_f32_16x16x4_f32, M = hidden, N = rows
//   a = sigma(z1), slope = a (1 - a) (as e^-z a^2), kept in registers in the
//       MFMA accumulator layout (lane: 1 row x 4 hidden units per 16x16 tile)
//   z2 = a W2^T + b2           per lane over its hidden units, then a
//                              reduce-scatter over the lanes of the row, so
//                              that lane (row n, group g) holds output g of
//                              row n and every lane evaluates one sigmoid
//   y = sigma(z2), delta2 = 2 (y - t) / (N K) . y (1 - y)
//   delta1^T = W2^T delta2^T   v_mfma_f32_16x16x4_f32 (the pre-update W2;
//                              the contraction over the <= 4 outputs is one
//                              instruction), times the slope
//   gW2^T += a^T delta2        v_mfma_f32_16x16x4_f32, K = the tile's rows
//   gW1 += delta1^T [X 1]      v_mfma_f32_16x16x4_f32, M = hidden, N = features,
//                              K = the tile's rows
//   gb2 += sum delta2          lane partials
//
// a, delta1 and delta2 pass through wave-private LDS tiles where a
// contraction needs them transposed.
//
// After a barrier the NW wave partials of every parameter are summed in wave
// order (bitwise repeatable) and the owner thread applies the update to the
// master copy in LDS, with its Kahan compensation term kept in registers;
// a second barrier publishes the new weights.  Padded rows carry zero X (so
// zero delta) and padded hidden units zero W2 (so zero delta1).
//
// Limits: N <= 128 rows, H <= 64, D <= 48, K <= 4.
#include <algorithm>
#include <type_traits>

#include "mlp_device.hpp"

namespace mlpk {

typedef float f32x4_s __attribute__((ext_vector_type(4)));

// The value of v in lane l of the wave (uniform result).
__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// LDS plan (floats).  The row count is the only size that is not fixed per
// kernel instance, so what depends on it comes last and every other address is
// a constant.
template <int NW, int HTM, int FT>
struct SmallPlan {
  static constexpr int HP = 16 * HTM;   // hidden units padded to 16-unit tiles
  static constexpr int DN = 16 * FT;    // features and the constant-1 column, padded to 16-wide tiles
  static constexpr int XS = DN + 2;     // row stride of X and W1: 16 rows of a tile hit distinct banks
  static constexpr int PW = HP * DN + 4 * HP + 4 + 4;   // one wave's partials: gW1 | gW2 | gb2 | loss
  static constexpr int w1 = 0;                  // [HP][XS] master W1|b1
  static constexpr int w2 = w1 + HP * XS;       // [4][HP]  master W2
  static constexpr int b2 = w2 + 4 * HP;        // [4]      master b2
  static constexpr int dst = b2 + 4;            // [NW][16][16] a staging (delta1's: in part)
  static constexpr int dd = dst + NW * 256;     // [NW][16][4] delta2 staging
  static constexpr int part = dd + NW * 64;     // [NW][PW] partials
  static constexpr int ts = part + NW * PW;     // [NP][4]  targets
  __host__ __device__ static int np(int n) { return (n + 15) / 16 * 16; }   // rows padded to 16-row tiles
  __host__ __device__ static int xs(int n) { return ts + np(n) * 4; }       // [NP][XS] rows
  __host__ __device__ static int vs(int n) { return xs(n) + np(n) * XS; }   // [P] velocity (momentum only)
};

// Training variants (the paper's method is act 0 without momentum):
// hidden activation act (0 sigma, 1 tanh); heavy-ball momentum with rate mu
// when vel (the velocity [P], packed order, of a single net) is not null.
struct SmallVariant {
  int act;
  float mu;
  float *vel;
};

// Four consecutive floats of LDS, 8-byte aligned.
__device__ __forceinline__ f32x4_s quad(const float *q) {
  const float2 lo = *reinterpret_cast<const float2 *>(q), hi = *reinterpret_cast<const float2 *>(q + 2);
  return f32x4_s{lo.x, lo.y, hi.x, hi.y};
}

// Waves per SIMD that the registers have to allow: two workgroups of 8 waves
// on a CU where the kernel is near 128 registers.  It matters above one net per
// CU, by launch hint (50 epochs with it and without: 472 nets of 120 x 30, 32 units
// 325 / 381 us, of 64 rows 225 / 282, of 120 x 20, 20 units, one output 285 / 350;
// 1000 nets of 120 x 30, 32 units 621 / 749) and costs nothing elsewhere (16 units
// 182 / 181; 15 features 238 / 241; 200 nets 190 / 190).
constexpr int small_waves(int nw, int htm, int ft) { return nw == 8 ? (htm <= 2 && ft <= 2 ? 4 : 2) : 1; }

// NW: waves; HTM: hidden tiles of the launch's widest net; FT: feature tiles
// (D + 1 columns); ACT: the hidden activation (0 sigma, 1 tanh).  Fixed per
// instance, so that LDS addresses are constants and nothing in the paper's
// sigmoid network branches for a variant.
template <int NW, int HTM, int FT, int ACT>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(small_waves(NW, HTM, FT)))) void k_small_train(
    const mlp_batch_item *__restrict__ items, mlp_batch_item one, int D, int K,
    const float *__restrict__ X, const float *__restrict__ T, float *__restrict__ theta,
    float *__restrict__ comp, int epochs, float *__restrict__ loss_hist, SmallVariant var) {
  using L = SmallPlan<NW, HTM, FT>;
  constexpr int NT = NW * 64;
  constexpr int PMAX = 16 * HTM * 16 * FT + 16 * HTM * 4 + 4;   // largest parameter count
  constexpr int JM = (PMAX + NT - 1) / NT;                      // parameters per thread
  constexpr int XS = L::XS, HP = L::HP, DN = L::DN, PW = L::PW, KO = 4;
  const mlp_batch_item it = items ? items[blockIdx.x] : one;
  const int N = it.n_rows, H = it.n_hidden;
  const float lr = it.lr;
  const int NP = L::np(N), NPT = NP / 16, HT = HTM == 1 ? 1 : (H + 15) / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;

  extern __shared__ float4 smem4[];
  float *sm = reinterpret_cast<float *>(smem4);
  float *Xs = sm + L::xs(N);
  float *W1s = sm + L::w1;
  float *W2s = sm + L::w2;
  float *b2s = sm + L::b2;
  float *Ts = sm + L::ts;
  float *Dst = sm + L::dst + wave * 256;
  float *Dd = sm + L::dd + wave * 64;
  float *Part = sm + L::part;
  float *Dst2 = Part + wave * PW;   // the wave's partials, free until they are written

  const float *Xg = X + it.x_off * D;
  const float *Tg = T + it.x_off * K;
  float *P = theta + it.p_off;
  float *Cp = comp ? comp + it.p_off : nullptr;
  const bool compensated = Cp != nullptr;
  const int D1 = D + 1;
  const int oB1 = H * D, oW2 = oB1 + H, oB2 = oW2 + K * H;
  const int nP = H * D1 + K * H + K;   // parameters, in update order: [W1 b1] rows, W2, b2

  // ---- stage rows, targets, parameters (coalesced); zero every padding entry
  for (int i = tid; i < NP * XS; i += NT) {
    const int r = i / XS, c = i - r * XS;
    Xs[i] = (r < N && c < D) ? Xg[(int64_t)r * D + c] : ((r < N && c == D) ? 1.0f : 0.0f);
  }
  for (int i = tid; i < NP * 4; i += NT) {
    const int r = i >> 2, k = i & 3;
    Ts[i] = (r < N && k < K) ? Tg[(int64_t)r * K + k] : 0.0f;
  }
  for (int i = tid; i < HP * XS; i += NT) {
    const int h = i / XS, c = i - h * XS;
    W1s[i] = (h < H && c < D) ? P[h * D + c] : ((h < H && c == D) ? P[oB1 + h] : 0.0f);
  }
  for (int i = tid; i < 4 * HP; i += NT) {
    const int k = i / HP, h = i - k * HP;
    W2s[i] = (k < K && h < H) ? P[oW2 + k * H + h] : 0.0f;
  }
  if (tid < 4) b2s[tid] = tid < K ? P[oB2 + tid] : 0.0f;
  // Kahan terms of the parameters this thread updates (q = tid + j*NT)
  // packed offset of parameter q (update order)
  auto packed = [&](int q) {
    if (q < H * D1) {
      const int h = q / D1, d = q - h * D1;
      return d < D ? h * D + d : oB1 + h;
    }
    if (q < H * D1 + K * H) return oW2 + (q - H * D1);
    return oB2 + (q - H * D1 - K * H);
  };
  float ccomp[JM];
#pragma unroll
  for (int j = 0; j < JM; ++j) {
    const int q = tid + j * NT;
    ccomp[j] = (compensated && q < nP) ? Cp[packed(q)] : 0.0f;
  }
  // momentum: the velocity lives in LDS in update order for the whole run
  float *Vs = sm + L::vs(N);
  if (var.vel)
    for (int q = tid; q < nP; q += NT) Vs[q] = var.vel[packed(q)];
  // LDS offsets of parameter q (update order): its partial within a wave's
  // block and its master copy.  Kept packed in registers across epochs when
  // a thread owns few parameters.
  auto offsets = [&](int q, int &po, int &mo) {
    if (q < H * D1) {
      const int h = q / D1, d = q - h * D1;
      // tile (h / 16, d / 16), lane (d % 16, h / 4 % 4), element h % 4
      po = ((h >> 4) * FT + (d >> 4)) * 256 + ((h >> 2 & 3) * 16 + (d & 15)) * 4 + (h & 3);
      mo = L::w1 + h * XS + d;
    } else if (q < H * D1 + K * H) {
      const int o = q - H * D1, k = o / H, h = o - k * H;
      po = HP * DN + k * HP + h;
      mo = L::w2 + k * HP + h;
    } else {
      const int k = q - H * D1 - K * H;
      po = HP * DN + 4 * HP + k;
      mo = L::b2 + k;
    }
  };
  constexpr bool kKeepOfs = JM <= 8;
  int uofs[kKeepOfs ? JM : 1];
  if constexpr (kKeepOfs) {
#pragma unroll
    for (int j = 0; j < JM; ++j) {
      const int q = tid + j * NT;
      int po = 0, mo = 0;
      if (q < nP) offsets(q, po, mo);
      uofs[j] = (po << 16) | mo;   // both below 2^16
    }
  }
  __syncthreads();

  const float dscale = 2.0f / (float)(N * K);
  const float inv_nk = 1.0f / (float)(N * K);

  // X operands of a row tile: of z1 (whole 16-feature groups) and of gW1 (rows
  // 4 s + lg).  With 8 waves most nets have a row tile per wave at most; the
  // operands then stay in registers for the run.
  f32x4_s xv[FT];
  float xb[FT][4];
  auto load_x = [&](int r0) {
    const float *xa = Xs + (r0 + l16) * XS + 4 * lg;
#pragma unroll
    for (int g = 0; g < FT; ++g) xv[g] = quad(xa + 16 * g);
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int s = 0; s < 4; ++s) xb[ft][s] = Xs[(r0 + lg + 4 * s) * XS + ft * 16 + l16];
  };
  const bool keep_x = NW == 8 && NPT <= NW;
  if (keep_x) load_x(min(wave, NPT - 1) * 16);

  for (int e = 0; e < epochs; ++e) {
    // ======================= rows of this wave: forward, deltas, partial gradients
    f32x4_s gacc[HTM][FT];   // gW1 tiles [hidden][feature]
    f32x4_s g2acc[HTM];     // gW2^T tiles [hidden][output]
#pragma unroll
    for (int ht = 0; ht < HTM; ++ht) {
      g2acc[ht] = f32x4_s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) gacc[ht][ft] = f32x4_s{0.f, 0.f, 0.f, 0.f};
    }
    float gb2 = 0.0f;   // output lg of this lane's rows
    float sq = 0.0f;

    for (int rt = wave; rt < NPT; rt += NW) {
      const int r0 = rt * 16;
      const int n = r0 + l16;   // this lane's row
      // z1^T tiles (M = hidden, N = rows): lane (row l16, group lg) holds
      // hidden units 4 lg .. 4 lg + 3 of each tile; a and its slope stay in
      // registers.  The contraction runs over whole 16-feature groups (the
      // padding is zero), index 4 lg + step within a group, so an operand of
      // four steps is one LDS read, and all of a tile's are issued ahead of
      // its products (one step at a time, each product waited for its own
      // reads: z1 and sigma took 1490 of a 60-row epoch's 5460 cycles).
      if (!keep_x) load_x(r0);
      const float b2k = b2s[lg], tk = Ts[n * 4 + lg];
      f32x4_s w2v[KO];   // one hidden tile: its W2 is read ahead of the products too (more: not enough registers)
      if (HTM == 1) {
#pragma unroll
        for (int k = 0; k < KO; ++k) w2v[k] = quad(W2s + k * HP + 4 * lg);
      }
      float av[HTM][4], sl[HTM][4];
#pragma unroll
      for (int ht = 0; ht < HTM; ++ht) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { av[ht][i] = 0.0f; sl[ht][i] = 0.0f; }
        if (ht < HT) {
          f32x4_s z = {0.f, 0.f, 0.f, 0.f}, wv[FT];
          const float *wb = W1s + (ht * 16 + l16) * XS + 4 * lg;
#pragma unroll
          for (int g = 0; g < FT; ++g) wv[g] = quad(wb + 16 * g);
#pragma unroll
          for (int g = 0; g < FT; ++g)
#pragma unroll
            for (int s = 0; s < 4; ++s) z = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[g][s], xv[g][s], z, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) av[ht][i] = ACT == 0 ? z[i] : hidden_act(ACT, z[i], sl[ht][i]);
          if (ACT == 0) {
            float ez[4];
            sigmoid_e4(av[ht], av[ht], ez);
#pragma unroll
            for (int i = 0; i < 4; ++i) sl[ht][i] = (ez[i] * av[ht][i]) * av[ht][i];
          }
        }
      }
      if (HTM == 1) {   // read by here, not one by one below
        asm volatile("" ::"v"(b2k), "v"(tk));
#pragma unroll
        for (int k = 0; k < KO; ++k) asm volatile("" ::"v"(w2v[k]));
      }
      // output layer: each lane's share of z2 (its 4 hidden units per tile)
      // for every output, then a reduce-scatter over the four row groups
      // (lanes n, n+16, n+32, n+48) leaves z2[n][lg] in lane (n, lg): every
      // lane evaluates one output of one row.  Padding hidden tiles read
      // tile 0's weights and multiply them by a zero activation.
      float zp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ht = 0; ht < HTM; ++ht) {
        const int hs = (ht < HT ? ht : 0) * 16 + 4 * lg;
#pragma unroll
        for (int k = 0; k < KO; ++k) {
          const f32x4_s w = HTM == 1 ? w2v[k] : quad(W2s + k * HP + hs);
#pragma unroll
          for (int i = 0; i < 4; ++i) zp[k] = fmaf(av[ht][i], w[i], zp[k]);
        }
      }
      const float z2 = add_swap16(add_swap32(zp[0], zp[2]), add_swap32(zp[1], zp[3]));
      const int k = lg;
      const float y = sigmoid(z2 + b2k);
      const bool on = k < K && n < N;
      const float err = on ? y - tk : 0.0f;
      sq = fmaf(err, err, sq);
      const float d2 = dscale * err * y * (1.0f - y);
      gb2 += d2;
      Dd[l16 * 4 + k] = d2;   // row-major [row][output] for the gW2 contraction
      float dv[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float v = Dd[(4 * s + lg) * 4 + (l16 & 3)];
        dv[s] = l16 < 4 ? v : 0.0f;
      }
#pragma unroll
      for (int ht = 0; ht < HTM; ++ht) {
        if (ht < HT) {
          // a and delta1 row-major through two LDS tiles of the wave (the
          // second one is its block of partials, free until they are
          // written), both written before either is read back:
          //   delta1^T = W2^T delta2^T (the pre-update W2), times the slope
          //   gW2^T += a^T delta2 (M = hidden, N = outputs, K = the tile's rows)
          //   gW1 += delta1^T [X 1]
          *reinterpret_cast<f32x4_s *>(Dst + l16 * 16 + 4 * lg) =
              f32x4_s{av[ht][0], av[ht][1], av[ht][2], av[ht][3]};
          const f32x4_s bp = __builtin_amdgcn_mfma_f32_16x16x4f32(
              W2s[lg * HP + ht * 16 + l16], d2, f32x4_s{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          *reinterpret_cast<f32x4_s *>(Dst2 + l16 * 16 + 4 * lg) =
              f32x4_s{bp[0] * sl[ht][0], bp[1] * sl[ht][1], bp[2] * sl[ht][2], bp[3] * sl[ht][3]};
          float ao[4], da[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) ao[s] = Dst[(4 * s + lg) * 16 + l16];
#pragma unroll
          for (int s = 0; s < 4; ++s) da[s] = Dst2[(4 * s + lg) * 16 + l16];
          f32x4_s g2 = g2acc[ht];
#pragma unroll
          for (int s = 0; s < 4; ++s) g2 = __builtin_amdgcn_mfma_f32_16x16x4f32(ao[s], dv[s], g2, 0, 0, 0);
          g2acc[ht] = g2;
          // (the feature tiles' chains interleave)
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int ft = 0; ft < FT; ++ft)
              gacc[ht][ft] = __builtin_amdgcn_mfma_f32_16x16x4f32(da[s], xb[ft][s], gacc[ht][ft], 0, 0, 0);
        }
      }
    }

    // ======================= wave partials to LDS
    float *pw = Part + wave * PW;
    // gW1 as the tiles lie in the lanes: 16 bytes a lane
    int lbase = 4 * lane;
    asm volatile("" : "+v"(lbase));   // addresses formed here, not held (or spilled) across the epoch loop
#pragma unroll
    for (int ht = 0; ht < HTM; ++ht) {
      if (ht < HT) {
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) *reinterpret_cast<f32x4_s *>(pw + lbase + (ht * FT + ft) * 256) = gacc[ht][ft];
        // lane (output l16, group lg): hidden units 4 lg .. 4 lg + 3
        if (l16 < 4) *reinterpret_cast<f32x4_s *>(pw + HP * DN + l16 * HP + ht * 16 + 4 * lg) = g2acc[ht];
      }
    }
    gb2 = sum16(gb2);
    if (l16 == 0) pw[HP * DN + 4 * HP + lg] = gb2;
    // (the lane reads stay outside the branch: the row sums must be complete
    // in all four rows, not only in the lane that stores)
    sq = sum16(sq);
    const float sqw = (lane_value(sq, 0) + lane_value(sq, 16)) + (lane_value(sq, 32) + lane_value(sq, 48));
    if (lane == 0) pw[HP * DN + 4 * HP + 4] = sqw;
    __syncthreads();

    // ======================= sum the wave partials in order; update
    if (loss_hist && tid == NT - 1) {   // (the last wave owns the fewest parameters)
      float s = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += Part[w * PW + HP * DN + 4 * HP + 4];
      loss_hist[(int64_t)blockIdx.x * epochs + e] = s * inv_nk;
    }
    if constexpr (kKeepOfs) {
      // the partial sums of a thread's first two parameters load
      // unconditionally (an unused slot reads offset 0), so both batches of
      // loads are in flight together
      float gs[JM];
#pragma unroll
      for (int j = 0; j < JM; ++j) {
        gs[j] = 0.0f;
        if (j < 2 || tid + j * NT < nP) {
          const int po = uofs[j] >> 16;
#pragma unroll
          for (int w = 0; w < NW; ++w) gs[j] += Part[w * PW + po];
        }
      }
#pragma unroll
      for (int j = 0; j < JM; ++j) {
        if (tid + j * NT < nP) {
          const int mo = uofs[j] & 0xffff;
          float wv = sm[mo], g = gs[j];
          if (var.vel) {   // heavy-ball momentum: v <- mu v + g, step along v
            g = fmaf(var.mu, Vs[tid + j * NT], g);
            Vs[tid + j * NT] = g;
          }
          gd_update(wv, ccomp[j], lr, g, compensated);
          sm[mo] = wv;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < JM; ++j) {
        const int q = tid + j * NT;
        if (q < nP) {
          int po, mo;
          offsets(q, po, mo);
          float g = 0.0f;
          for (int w = 0; w < NW; ++w) g += Part[w * PW + po];
          if (var.vel) {
            g = fmaf(var.mu, Vs[q], g);
            Vs[q] = g;
          }
          float wv = sm[mo];
          gd_update(wv, ccomp[j], lr, g, compensated);
          sm[mo] = wv;
        }
      }
    }
    __syncthreads();
  }

  // ---- write the trained parameters (and compensation) back once
#pragma unroll
  for (int j = 0; j < JM; ++j) {
    const int q = tid + j * NT;
    if (q < nP) {
      int o;
      float wv;
      if (q < H * D1) {
        const int h = q / D1, d = q - h * D1;
        o = d < D ? h * D + d : oB1 + h;
        wv = W1s[h * XS + d];
      } else if (q < H * D1 + K * H) {
        const int oo = q - H * D1, k = oo / H, h = oo - k * H;
        o = oW2 + oo;
        wv = W2s[k * HP + h];
      } else {
        const int k = q - H * D1 - K * H;
        o = oB2 + k;
        wv = b2s[k];
      }
      P[o] = wv;
      if (compensated) Cp[o] = ccomp[j];
    }
  }
  if (var.vel)
    for (int q = tid; q < nP; q += NT) var.vel[packed(q)] = Vs[q];
}

// The instance for a launch's waves, widest net, features and activation.
template <int NW, int ACT, int HTM = 1, int FT = 1>
const void *small_kernel(int ht, int ft) {
  if (ht == HTM && ft == FT) return (const void *)k_small_train<NW, HTM, FT, ACT>;
  if constexpr (HTM < 4) {
    if (ht > HTM) return small_kernel<NW, ACT, HTM + 1, FT>(ht, ft);
  }
  if constexpr (FT < 4) return small_kernel<NW, ACT, HTM, FT + 1>(ht, ft);
  return nullptr;
}

// ---------------------------------------------------------------------------
// Hidden-split form of the same trainer (the paper's sigmoid network, plain
// or compensated update): the NW waves of a workgroup split the hidden layer
// instead of the rows.  Wave w owns hidden tile w (units 16 w .. 16 w + 15)
// for every row of the net; waves past the net's last tile only pass the
// barriers.  Per epoch:
//   phase A (every 16-row tile): z1^T of the wave's tile on MFMA, e^-z1 kept
//     in registers for the epoch, and the tile's share of z2 (its
//     16 hidden units, reduce-scattered over the lanes of a row) to LDS;
//   one barrier;
//   phase B (every row tile): z2 = the tiles' shares summed in tile order
//     plus b2, y and delta2 (each wave forms them itself, so every wave holds
//     the same values), then for the wave's own units a and the slope again
//     from e^-z1 (a reciprocal; holding both would take 32 more registers and
//     a third of the resident nets),
//     gW2 += a^T delta2,
//     delta1 = (W2^T delta2) . slope with the pre-update W2, and
//     gW1 += delta1^T [X 1], all on MFMA and accumulated in registers;
//   the update: each wave applies its own W1 rows and W2 columns from the
//     registers that hold their gradients, the Kahan terms living in the same
//     lanes; b2 is kept and updated in registers by every wave alike (the
//     same delta2 sums), wave 0 writing it back at the end.
// A wave reads only its own W1 rows and W2 columns, the shares of consecutive
// epochs alternate between two buffers, and b2 is private to each wave, so
// one barrier per epoch suffices and no per-wave partial gradients exist:
// LDS holds X, the parameters and the shares only (the targets of a lane's
// rows stay in its registers for the run).  The row stride of X and W1 is
// the z1 contraction's length: the gW1 operand of the feature block past it
// reads into the next row, which only feeds gradients of padding
// features that are never applied; so three 120-row, 64-unit nets share a CU.
// Limits: N <= 128 rows, H <= 16 NW <= 64, D <= 48, K <= KO <= 4.
struct HSplitLayout {
  int NP, HP, XS, NW, KO;
  __host__ __device__ HSplitLayout(int n, int h, int d, int nw, int ko)
      : NP((n + 15) / 16 * 16), HP((h + 15) / 16 * 16), XS(row_stride(steps(d))), NW(nw), KO(ko) {}
  __host__ __device__ static constexpr int steps(int d) { return (d + 1 + 3) / 4; }
  // an odd multiple of 4: the 16 rows x 4 features of a z1 operand lie in 64 banks
  __host__ __device__ static constexpr int row_stride(int ks) { return 4 * (ks | 1); }
  __host__ __device__ int xs() const { return 0; }                 // [NP][XS] rows, ones column
  __host__ __device__ int w1() const { return xs() + NP * XS; }    // [HP][XS] W1 | b1
  __host__ __device__ int w2() const { return w1() + HP * XS; }    // [4][64]
  __host__ __device__ int zs() const { return w2() + 256; }        // [2][NW][NP][KO] z2 shares
  __host__ __device__ int dst() const { return (zs() + 2 * NW * NP * KO + 3) / 4 * 4; }   // [NW][2][16][16] staging
  __host__ __device__ int dd() const { return dst() + NW * 512; }  // [NW][2][16][4] delta2 staging
  __host__ __device__ int total() const { return dd() + NW * 128 + 64; }   // + the over-read of the last X row
};

// At most 168 registers per lane (three waves per SIMD): three nets of 120 rows,
// 64 units and 33 features (51 KB of LDS each) share a CU.
// The contraction's length is a template size (KS steps of 4 features), so
// every LDS address is a lane's base and an immediate.  Bound: the SIMDs'
// float32 units, which products and vector work share: 1450 nets of up to 120
// rows and 64 units have the matrix cores busy 37 % of the cycles and the vector
// unit 41 %, 8.2 vector instructions a product.  With run-time strides they were
// nine, a third of them addresses and branches (4096 networks on this form, 100
// epochs: 8.1 ms, now 6.0).
template <int KS, int KO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_small_hsplit(
    const mlp_batch_item *__restrict__ items, mlp_batch_item one, int D, int K,
    const float *__restrict__ X, const float *__restrict__ T, float *__restrict__ theta,
    float *__restrict__ comp, int epochs, float *__restrict__ loss_hist) {
  constexpr int XS = HSplitLayout::row_stride(KS), FT = (KS + 3) / 4, WS2 = 64;   // WS2: row stride of W2
  const int NT = blockDim.x, NW = NT >> 6;
  const mlp_batch_item it = items ? items[blockIdx.x] : one;
  const int N = it.n_rows, H = it.n_hidden;
  const float lr = it.lr;
  const HSplitLayout L(N, H, D, NW, KO);
  const int HP = L.HP, NP = L.NP, NPT = NP / 16;
  const int HTn = HP / 16;   // hidden tiles of this net
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16_0 = lane & 15, lg_0 = lane >> 4;
  int l16 = l16_0, lg = lg_0;

  extern __shared__ float4 smem4[];
  float *sm = reinterpret_cast<float *>(smem4);
  float *Xs = sm + L.xs();
  float *W1s = sm + L.w1();
  float *W2s = sm + L.w2();
  float *Zs = sm + L.zs();
  float *Dst = sm + L.dst() + wave * 512;   // two buffers: a pair of row tiles
  float *Dd = sm + L.dd() + wave * 128;

  const float *Xg = X + it.x_off * D;
  const float *Tg = T + it.x_off * K;
  float *P = theta + it.p_off;
  float *Cp = comp ? comp + it.p_off : nullptr;
  const bool compensated = Cp != nullptr;
  const int D1 = D + 1;
  const int oB1 = H * D, oW2 = oB1 + H, oB2 = oW2 + K * H;

  // ---- stage rows (with the ones column), targets, W1 | b1, W2; zero padding
  for (int i = tid; i < NP * XS; i += NT) {
    const int r = i / XS, c = i - r * XS;
    Xs[i] = (r < N && c < D) ? Xg[(int64_t)r * D + c] : ((r < N && c == D) ? 1.0f : 0.0f);
  }
  for (int i = tid; i < HP * XS; i += NT) {
    const int h = i / XS, c = i - h * XS;
    W1s[i] = (h < H && c < D) ? P[h * D + c] : ((h < H && c == D) ? P[oB1 + h] : 0.0f);
  }
  // the target of lane (row l16, output lg) of every row tile
  float tv[8];
#pragma unroll
  for (int rt = 0; rt < 8; ++rt) {
    const int n = rt * 16 + l16;
    tv[rt] = (n < N && lg < K) ? Tg[(int64_t)n * K + lg] : 0.0f;
  }
  for (int i = tid; i < 4 * WS2; i += NT) {
    const int k = i / WS2, h = i - k * WS2;
    W2s[i] = (k < K && h < H) ? P[oW2 + k * H + h] : 0.0f;
  }
  // this wave's tile and the parameters its lanes update: W1[h0 + 4 lg + i]
  // [16 ft + l16] (b1 is column D), W2[l16][h0 + 4 lg + i] for l16 < K, and
  // b2[lg] (every wave's own copy)
  const bool own = wave < HTn;
  const int h0 = wave * 16;
  float c1[FT][4], c2[4];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = h0 + 4 * lg + i, d = 16 * ft + l16;
      c1[ft][i] = (compensated && own && h < H && d < D1) ? Cp[d < D ? h * D + d : oB1 + h] : 0.0f;
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int h = h0 + 4 * lg + i;
    c2[i] = (compensated && own && l16 < K && h < H) ? Cp[oW2 + l16 * H + h] : 0.0f;
  }
  float b2v = lg < K ? P[oB2 + lg] : 0.0f;
  float cb = (compensated && lg < K) ? Cp[oB2 + lg] : 0.0f;
  __syncthreads();

  const float dscale = 2.0f / (float)(N * K);
  const float inv_nk = 1.0f / (float)(N * K);

  for (int e = 0; e < epochs; ++e) {
    float *zs = Zs + (e & 1) * (NW * NP * KO) + l16_0 * KO + lg_0;   // this lane's share in wave 0's row tile 0
    // the lane coordinates, opaque to the compiler each epoch: the per-lane
    // LDS addresses are formed here instead of being hoisted out of the
    // epoch loop and held (or spilled) for the whole run
    int l16 = l16_0, lg = lg_0;
    asm volatile("" : "+v"(l16), "+v"(lg));
    float ez[8][4];   // e^-z1 of this wave's units, every row tile (a and the slope are re-formed from it)
    const int ZW = NP * KO;   // z2 shares of a wave
    // ======================= phase A: a of this wave's tile, its share of z2
    // Row tiles go in pairs whose two z1 chains share the W1 operand and
    // interleave on the matrix cores (a lone last tile runs its own chain).
    if (own) {
      const float *wb = W1s + (h0 + l16) * XS + lg;
      float w[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) w[s] = wb[4 * s];
      f32x4_s w2v[KO];
#pragma unroll
      for (int k = 0; k < KO; ++k) w2v[k] = *reinterpret_cast<const f32x4_s *>(W2s + k * WS2 + h0 + 4 * lg);
      auto finish = [&](auto rt_c, const f32x4_s &z) {
        constexpr int rt = decltype(rt_c)::value;
        float a[4] = {z[0], z[1], z[2], z[3]};
        sigmoid_e4(a, a, ez[rt]);
        float zp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KO; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i) zp[k] = fmaf(a[i], w2v[k][i], zp[k]);
        // reduce-scatter over the row's four lane groups: lane (row, lg)
        // ends with output lg of the row
        const float share = add_swap16(add_swap32(zp[0], zp[2]), add_swap32(zp[1], zp[3]));
        if (lg < KO) zs[wave * ZW + rt * 16 * KO] = share;
      };
      auto pair = [&](auto r0_c) {
        constexpr int r0 = decltype(r0_c)::value;
        const float *xa = Xs + (r0 * 16 + l16) * XS + lg;
        if (r0 + 1 < NPT) {
          const float *xb = xa + 16 * XS;
          f32x4_s za = {0.f, 0.f, 0.f, 0.f}, zb = {0.f, 0.f, 0.f, 0.f};
          float a[KS], b[KS];   // read ahead of the products
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            a[s] = xa[4 * s];
            b[s] = xb[4 * s];
          }
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            za = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], a[s], za, 0, 0, 0);
            zb = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], b[s], zb, 0, 0, 0);
          }
          finish(std::integral_constant<int, r0>{}, za);
          finish(std::integral_constant<int, r0 + 1>{}, zb);
        } else if (r0 < NPT) {
          f32x4_s za = {0.f, 0.f, 0.f, 0.f};
          float a[KS];
#pragma unroll
          for (int s = 0; s < KS; ++s) a[s] = xa[4 * s];
#pragma unroll
          for (int s = 0; s < KS; ++s) za = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s], a[s], za, 0, 0, 0);
          finish(std::integral_constant<int, r0>{}, za);
        }
      };
      pair(std::integral_constant<int, 0>{});
      pair(std::integral_constant<int, 2>{});
      pair(std::integral_constant<int, 4>{});
      pair(std::integral_constant<int, 6>{});
    }
    __syncthreads();
    if (!own) continue;
    // ======================= phase B: delta2, then this tile's gradients
    // Row tiles again go in pairs (two staging buffers); a pair's products
    // start from zero and are added to the totals, so a gradient of 128 rows is
    // 32 + 4 roundings deep and not one chain of 128 (128 rows of 48-64-3: rms
    // error of a step's gradients 17.8e-9 of the largest, so 8.6e-9; on 2 waves
    // that split the rows 11.2e-9.  4096 networks 5310 -> 5375 us.)
    f32x4_s gacc[FT], g2 = {0.f, 0.f, 0.f, 0.f};
    f32x4_s part = {0.f, 0.f, 0.f, 0.f}, parts[FT];   // of the last pair, added under the next one's loads
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) gacc[ft] = parts[ft] = f32x4_s{0.f, 0.f, 0.f, 0.f};
    auto add_parts = [&]() {
      g2 += part;
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) gacc[ft] += parts[ft];
    };
    float gb2 = 0.0f, sq = 0.0f;
    // delta2 of row tile rt in lane (row l16, output lg)
    auto delta2 = [&](auto rt_c) {
      constexpr int rt = decltype(rt_c)::value;
      const int n = rt * 16 + l16, k = lg;
      float z2 = 0.0f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {   // (a share past the net's last wave: its own last one, adding zero)
        const float share = zs[min(w, HTn - 1) * ZW + rt * 16 * KO];
        z2 += w < HTn ? share : 0.0f;
      }
      if (k >= KO) z2 = 0.0f;   // no output: another row's share
      const float y = sigmoid(z2 + b2v);
      const bool on = k < K && n < N;
      const float err = on ? y - tv[rt] : 0.0f;
      sq = fmaf(err, err, sq);
      const float d2 = dscale * err * y * (1.0f - y);
      gb2 += d2;
      return d2;
    };
    // the gradients of NR (1 or 2) consecutive row tiles from r0
    auto tiles = [&](auto r0_c, auto nr_c) {
      constexpr int r0 = decltype(r0_c)::value, NR = decltype(nr_c)::value;
      float d2[NR];
      d2[0] = delta2(std::integral_constant<int, r0>{});
      if constexpr (NR == 2) d2[NR - 1] = delta2(std::integral_constant<int, r0 + 1>{});
      float av[NR][4], sl[NR][4];
#pragma unroll
      for (int j = 0; j < NR; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) av[j][i] = sigmoid_slope_of_e(ez[r0 + j][i], sl[j][i]);
        Dd[j * 64 + l16 * 4 + lg] = d2[j];
        *reinterpret_cast<f32x4_s *>(Dst + j * 256 + l16 * 16 + 4 * lg) = f32x4_s{av[j][0], av[j][1], av[j][2], av[j][3]};
      }
      // gW2^T += a^T delta2 (M = hidden, N = outputs, K = the tile's rows)
      add_parts();
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float dv = Dd[j * 64 + (4 * s + lg) * 4 + (l16 & 3)];
          part = __builtin_amdgcn_mfma_f32_16x16x4f32(Dst[j * 256 + (4 * s + lg) * 16 + l16], l16 < 4 ? dv : 0.0f,
                                                     j || s ? part : f32x4_s{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
      // delta1^T = W2^T delta2^T (the pre-update W2), times the slope
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const f32x4_s bp = __builtin_amdgcn_mfma_f32_16x16x4f32(W2s[lg * WS2 + h0 + l16], d2[j],
                                                               f32x4_s{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        *reinterpret_cast<f32x4_s *>(Dst + j * 256 + l16 * 16 + 4 * lg) =
            f32x4_s{bp[0] * sl[j][0], bp[1] * sl[j][1], bp[2] * sl[j][2], bp[3] * sl[j][3]};
      }
      // gW1 += delta1^T [X 1] (M = hidden, N = features, K = the tile's rows)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        float da[4], xb[FT][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          da[s] = Dst[j * 256 + (lg + 4 * s) * 16 + l16];
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) xb[ft][s] = Xs[((r0 + j) * 16 + lg + 4 * s) * XS + ft * 16 + l16];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int ft = 0; ft < FT; ++ft)
            parts[ft] = __builtin_amdgcn_mfma_f32_16x16x4f32(da[s], xb[ft][s],
                                                             j || s ? parts[ft] : f32x4_s{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      }
    };
    auto pair_b = [&](auto r0_c) {
      constexpr int r0 = decltype(r0_c)::value;
      if (r0 + 1 < NPT) tiles(r0_c, std::integral_constant<int, 2>{});
      else if (r0 < NPT) tiles(r0_c, std::integral_constant<int, 1>{});
    };
    pair_b(std::integral_constant<int, 0>{});
    pair_b(std::integral_constant<int, 2>{});
    pair_b(std::integral_constant<int, 4>{});
    pair_b(std::integral_constant<int, 6>{});
    add_parts();
    if (wave == 0 && loss_hist) {
      const float sqw = wave_sum(sq);
      if (lane == 0) loss_hist[(int64_t)blockIdx.x * epochs + e] = sqw * inv_nk;
    }
    // ======================= update: this wave's W1 rows and W2 columns, b2
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = h0 + 4 * lg + i;
      if (h < H) {
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) {
          if (ft < FT - 1 || 16 * ft + l16 < D1) {
            float *wp = W1s + (h0 + 4 * lg) * XS + l16 + i * XS + 16 * ft;
            float wv = *wp;
            gd_update(wv, c1[ft][i], lr, gacc[ft][i], compensated);
            *wp = wv;
          }
        }
      }
    }
    if (l16 < K) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int h = h0 + 4 * lg + i;
        if (h < H) {
          const int o = l16 * WS2 + h;
          float wv = W2s[o];
          gd_update(wv, c2[i], lr, g2[i], compensated);
          W2s[o] = wv;
        }
      }
    }
    // every lane of group lg holds the row sum of output lg after sum16
    gb2 = sum16(gb2);
    if (lg < K) gd_update(b2v, cb, lr, gb2, compensated);
  }
  __syncthreads();

  // ---- write the trained parameters (and compensation) back once
  if (own) {
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int h = h0 + 4 * lg + i, d = 16 * ft + l16;
        if (h < H && d < D1) {
          const int o = d < D ? h * D + d : oB1 + h;
          P[o] = W1s[h * XS + d];
          if (compensated) Cp[o] = c1[ft][i];
        }
      }
    }
    if (l16 < K) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int h = h0 + 4 * lg + i;
        if (h < H) {
          P[oW2 + l16 * H + h] = W2s[l16 * WS2 + h];
          if (compensated) Cp[oW2 + l16 * H + h] = c2[i];
        }
      }
    }
  }
  if (wave == 0 && l16 == 0 && lg < K) {
    P[oB2 + lg] = b2v;
    if (compensated) Cp[oB2 + lg] = cb;
  }
}

// The instance for KS steps of 4 features (n_in <= 48 and the constant column).
template <int KO, int KS = 13>
const void *hsplit_kernel(int steps) {
  if constexpr (KS > 1) {
    if (steps < KS) return hsplit_kernel<KO, KS - 1>(steps);
  }
  return reinterpret_cast<const void *>(&k_small_hsplit<KS, KO>);
}

}  // namespace mlpk

namespace mlph {

size_t small_lds_bytes(int n_rows, int n_hidden, int n_in, int threads, bool momentum) {
  const int nw = threads / 64, ht = (n_hidden + 15) / 16, ft = (n_in + 16) / 16, np = (n_rows + 15) / 16 * 16;
  const int hp = 16 * ht, dn = 16 * ft;   // SmallPlan's, for run-time sizes
  const int pw = hp * dn + 4 * hp + 8;
  const int mom = momentum ? (n_hidden * (n_in + 1) + 4 * n_hidden + 4 + 3) / 4 * 4 : 0;
  return sizeof(float) * (size_t)(hp * (dn + 2) + 4 * hp + 4 + nw * (256 + 64 + pw) + np * (4 + dn + 2) + mom);
}

// Launch shape of n_nets nets of at most max_hidden units (0: no hint).  Up
// to one net per CU a net's own epoch counts: 8 waves (86 nets of 120 rows x
// 63 units, 20 epochs: 170 us against 220 on 4 waves, 206 hidden-split).
// Above, the chip is shared and the work of a net counts: hidden-split over
// 32 units (1450 nets of 120 rows x 64 units: 804 us against 1014 on 8 waves,
// 1227 on 2 and 1312 on 4), else 4 waves (1465 nets of 32 units: 472 us
// against 555 on 8, 582 hidden-split; 2759 of 16: 428, 455, 701).
int small_threads(int n_nets, int max_hidden, int n_cu, int hint) {
  if (hint == kHiddenSplit || hint == 128 || hint == 256 || hint == 512) return hint;
  if (n_nets <= n_cu) return 512;
  return max_hidden > 32 ? kHiddenSplit : 256;
}

size_t small_launch_lds_bytes(int max_rows, int max_hidden, int n_in, int threads, bool momentum) {
  // the layout grows monotonically with N and H
  return small_lds_bytes(max_rows, max_hidden, n_in, threads, momentum);
}

hipError_t launch_small_train(const mlp_batch_item *items, mlp_batch_item one, int n_nets,
                              int n_in, int n_out, int max_rows, int max_hidden, const float *X,
                              const float *T, float *theta, float *comp, int epochs,
                              float *loss_hist, int act, float mu, float *vel, int threads, hipStream_t s) {
  const mlpk::SmallVariant var{act, mu, vel};
  const bool mom = vel != nullptr;
  if (threads == kHiddenSplit) {
    if (act == 0 && !mom) {
      // one wave per 16 hidden units of the launch's widest net
      const int tiles = (max_hidden + 15) / 16;
      const int nw = tiles <= 1 ? 1 : (tiles <= 2 ? 2 : 4);
      const size_t lds =
          sizeof(float) * (size_t)mlpk::HSplitLayout(max_rows, max_hidden, n_in, nw, n_out <= 3 ? 3 : 4).total();
      const int steps = mlpk::HSplitLayout::steps(n_in);
      const void *kern = n_out <= 3 ? mlpk::hsplit_kernel<3>(steps) : mlpk::hsplit_kernel<4>(steps);
      hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      void *args[] = {&items, &one, &n_in, &n_out, &X, &T, &theta, &comp, &epochs, &loss_hist};
      e = hipLaunchKernel(kern, dim3(n_nets), dim3(64 * nw), args, lds, s);
      return e == hipSuccess ? hipGetLastError() : e;
    }
    threads = 128;   // the variants run on the row-split form
  }
  // fewer waves when the per-wave partial buffers would not fit in LDS
  while (threads > 128 && small_launch_lds_bytes(max_rows, max_hidden, n_in, threads, mom) > 160 * 1024)
    threads /= 2;
  const size_t lds = small_launch_lds_bytes(max_rows, max_hidden, n_in, threads, mom);
  // the tanh variant is instantiated for 8 waves only; the host API checks
  // that its LDS plan fits before launching
  if (act == 1 && threads != 512) return hipErrorInvalidValue;
  const int ht = (max_hidden + 15) / 16, ft = (n_in + 16) / 16;   // (the constant column is a feature)
  const void *kern = act == 1         ? mlpk::small_kernel<8, 1>(ht, ft)
                     : threads == 512 ? mlpk::small_kernel<8, 0>(ht, ft)
                     : threads == 256 ? mlpk::small_kernel<4, 0>(ht, ft)
                                      : mlpk::small_kernel<2, 0>(ht, ft);
  hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  mlpk::SmallVariant v = var;
  void *args[] = {&items, &one, &n_in, &n_out, &X, &T, &theta, &comp, &epochs, &loss_hist, &v};
  e = hipLaunchKernel(kern, dim3(n_nets), dim3(threads), args, lds, s);
  return e == hipSuccess ? hipGetLastError() : e;
}

}  // namespace mlph
