// Fused full-batch trainer for networks with several hidden layers: section
// 2.2's loop (feed forward layer by layer, the error, backpropagation from
// the top layer down, every layer's update) for L weight layers, the whole
// run in one launch of one workgroup with the rows, targets, activations,
// deltas and parameters resident in LDS.
//
// Per epoch, separated by workgroup barriers:
//   forward, one phase per layer: lane (row r, units o and o + half) forms
//     z = b_l[o] + sum_i A_l[r][i] W_l[o][i] and applies the hidden
//     activation (the sigmoid of Equation 1 or tanh) or, on the top layer,
//     the sigmoid; rows are the fast index across lanes, so the weight row
//     is a broadcast read and the activation rows (odd strides) hit
//     distinct banks;
//   error: the mean squared error's terms and the top delta
//     2 (y - t) / (n K) * y (1 - y), the loss summed wave by wave in a
//     fixed order;
//   backward, one phase per layer, top down: the gradient of W_l and b_l as
//     sums over rows split into RS fixed row segments (one partial per
//     segment, so several lanes share a long sum), and, below the top layer,
//     the delta of the layer below through the pre-update W_l times the
//     slope of its activation;
//   update: the RS partials of each parameter added in segment order, then
//   theta <- theta - lr g (Kahan-compensated when a compensation array is
//   given) for every layer at once.
// All sums run in fixed orders, so a run is bitwise repeatable.
#include <algorithm>

#include "deep.hpp"
#include "mlp_device.hpp"

namespace mlpk {

using mlph::DeepPlan;

// x / d and x mod d for 0 <= x < 2^20, 1 <= d, from the float reciprocal
// inv = 1/d: the estimate is within one of the quotient (relative error
// below 2^-22 on a quotient below 2^20) and one correction step makes it
// exact.  About eight VALU operations instead of an integer division.
__device__ __forceinline__ int div_small(int x, int d, float inv, int &rem) {
  int q = (int)((float)x * inv);
  int r = x - q * d;
  if (r < 0) {
    q -= 1;
    r += d;
  } else if (r >= d) {
    q += 1;
    r -= d;
  }
  rem = r;
  return q;
}

template <int ACT>
__global__ __launch_bounds__(mlph::kDeepThreads) void k_deep_train(
    DeepPlan p, const float *__restrict__ X, const float *__restrict__ T, float *__restrict__ theta,
    float *__restrict__ comp, float lr, int epochs, float *__restrict__ loss_hist) {
  constexpr int NT = mlph::kDeepThreads, NW = NT / kWave;
  extern __shared__ float4 smem4[];
  float *sm = reinterpret_cast<float *>(smem4);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int L = p.L, n = p.n, P = p.P, K = p.w[L], sK = p.sa[L], sd = p.sd;
  const bool compensated = comp != nullptr;

  // ---- stage rows, targets, parameters and compensation terms (coalesced)
  {
    const int d = p.w[0], s = p.sa[0];
    for (int i = tid; i < n * d; i += NT) {
      const int r = i / d, c = i - r * d;
      sm[p.aoff[0] + r * s + c] = X[i];
    }
  }
  for (int i = tid; i < n * K; i += NT) {
    const int r = i / K, k = i - r * K;
    sm[p.toff + r * sK + k] = T[i];
  }
  // a column of ones after every layer input's row: the bias is the last
  // column of the gradient's row sums
  for (int i = tid; i < n * L; i += NT) {
    const int l = i / n, r = i - l * n;
    sm[p.aoff[l] + r * p.sa[l] + p.w[l]] = 1.0f;
  }
  for (int q = tid; q < P; q += NT) {
    sm[p.th + q] = theta[q];
    sm[p.cp + q] = compensated ? comp[q] : 0.0f;
  }
  __syncthreads();

  const float dscale = 2.0f / ((float)n * (float)K);
  const float inv_nk = 1.0f / ((float)n * (float)K);
  float *Dtop = sm + ((L & 1) ? p.d1 : p.d0);

  for (int e = 0; e < epochs; ++e) {
    // ======================= feed forward
    for (int l = 0; l < L; ++l) {
      const int wi = p.w[l], wo = p.w[l + 1], si = p.sa[l], so = p.sa[l + 1];
      const float *A = sm + p.aoff[l];
      const float *W = sm + p.th + p.poff[l];
      const float *b = W + wo * wi;
      float *Y = sm + p.aoff[l + 1];
      const bool hidden = l < L - 1;
      // units in pairs (o0, o0 + hO) of one row: the row's inputs load once
      const int hO = (wo + 1) >> 1;
      const float inv_n = 1.0f / (float)n;
      for (int idx = tid; idx < n * hO; idx += NT) {
        int r;
        const int o0 = div_small(idx, n, inv_n, r);
        const int o1 = o0 + hO, o1r = min(o1, wo - 1);   // o1 = wo only when wo is odd: dropped
        const float *a = A + r * si, *w0 = W + o0 * wi, *w1 = W + o1r * wi;
        float z0 = b[o0], z1 = b[o1r];
#pragma unroll 8
        for (int i = 0; i < wi; ++i) {
          const float av = a[i];
          z0 = fmaf(av, w0[i], z0);
          z1 = fmaf(av, w1[i], z1);
        }
        Y[r * so + o0] = (hidden && ACT == 1) ? tanhf(z0) : sigmoid(z0);
        if (o1 < wo) Y[r * so + o1] = (hidden && ACT == 1) ? tanhf(z1) : sigmoid(z1);
      }
      __syncthreads();
    }

    // ======================= error and the top layer's delta
    {
      const float *Y = sm + p.aoff[L], *Ts = sm + p.toff;
      float part = 0.0f;
      const float inv_k = 1.0f / (float)K;
      for (int idx = tid; idx < n * K; idx += NT) {
        int k;
        const int r = div_small(idx, K, inv_k, k);
        const float y = Y[r * sK + k], d = y - Ts[r * sK + k];
        part = fmaf(d, d, part);
        Dtop[r * sd + k] = (dscale * d) * (y * (1.0f - y));
      }
      part = wave_sum(part);
      if (lane == 0) sm[p.red + wave] = part;
      __syncthreads();
      if (loss_hist && tid == 0) {
        float t = 0.0f;
        for (int w = 0; w < NW; ++w) t += sm[p.red + w];
        loss_hist[e] = t * inv_nk;
      }
    }

    // ======================= backpropagation, top layer first
    for (int l = L - 1; l >= 0; --l) {
      const int wi = p.w[l], wo = p.w[l + 1], si = p.sa[l];
      const float *A = sm + p.aoff[l];
      const float *W = sm + p.th + p.poff[l];
      const float *Dn = sm + (((l + 1) & 1) ? p.d1 : p.d0);
      float *Dl = sm + ((l & 1) ? p.d1 : p.d0);
      // the gradient's columns c = 0 .. wi (c = wi: the bias) in pairs (c, c + h)
      const int h = (wi + 2) >> 1, nW = wo * h, nG = p.RS * nW, nD = l > 0 ? n * wi : 0;
      float *G = sm + p.gr + p.poff[l];
      const float inv_nw = 1.0f / (float)nW, inv_h = 1.0f / (float)h, inv_wi = 1.0f / (float)wi;
      for (int idx = tid; idx < nG + nD; idx += NT) {
        if (idx < nG) {
          // segment sg of the row sums of parameters (o, c0) and (o, c1);
          // column wi is the bias (its input is the column of ones)
          int k, c0;
          const int sg = div_small(idx, nW, inv_nw, k);
          const int o = div_small(k, h, inv_h, c0);
          const int c1 = c0 + h, c1r = min(c1, wi);   // c1 = wi + 1 only when wi + 1 is odd: dropped
          const int r0 = sg * p.seg, r1 = min(n, r0 + p.seg);
          float acc0 = 0.0f, acc1 = 0.0f;
#pragma unroll 8
          for (int r = r0; r < r1; ++r) {
            const float d = Dn[r * sd + o];
            const float *ar = A + r * si;
            acc0 = fmaf(d, ar[c0], acc0);
            acc1 = fmaf(d, ar[c1r], acc1);
          }
          G[sg * P + (c0 < wi ? o * wi + c0 : wo * wi + o)] = acc0;
          if (c1 <= wi) G[sg * P + (c1 < wi ? o * wi + c1 : wo * wi + o)] = acc1;
        } else {
          // delta of layer l's input units (a hidden layer) at row r
          const int j = idx - nG;
          int i;
          const int r = div_small(j, wi, inv_wi, i);
          const float *dr = Dn + r * sd;
          float acc = 0.0f;
#pragma unroll 8
          for (int o = 0; o < wo; ++o) acc = fmaf(dr[o], W[o * wi + i], acc);
          const float a = A[r * si + i];
          Dl[r * sd + i] = acc * (ACT == 1 ? 1.0f - a * a : a * (1.0f - a));
        }
      }
      __syncthreads();
    }

    // ======================= update every layer at once
    for (int q = tid; q < P; q += NT) {
      float g = sm[p.gr + q];
      for (int sg = 1; sg < p.RS; ++sg) g += sm[p.gr + sg * P + q];
      float w = sm[p.th + q], c = sm[p.cp + q];
      gd_update(w, c, lr, g, compensated);
      sm[p.th + q] = w;
      sm[p.cp + q] = c;
    }
    __syncthreads();
  }

  // ---- write the trained parameters (and compensation) back once
  for (int q = tid; q < P; q += NT) {
    theta[q] = sm[p.th + q];
    if (compensated) comp[q] = sm[p.cp + q];
  }
}

// ---------------------------------------------------------------------------
// The same training loop on the matrix cores (v_mfma_f32_16x16x4_f32), for two
// to four layers with outputs of up to 64 units (at most 16 of the top layer).
// An epoch has two parts, each ended by a barrier:
//   rows: every wave takes its 16-row tiles through all layers, forward and
//     back (rows do not interact):
//       z^T = W a^T            M = units, N = rows: a lane holds one row and
//                              four units of a tile, which are the next
//                              layer's (and the delta's) operands as they lie,
//                              the contraction index running over 4 lg + step;
//                              b starts the accumulator
//       delta_l-1^T = W^T delta_l^T . slope      the same way, downwards
//     and leaves activations and deltas in LDS;
//   weights: every wave owns 16 x 16 tiles of the weights, sums
//       gW = delta^T a         M = units, N = inputs, K = all rows
//     (and gb) in its registers and updates the tile in place.
// Unit counts are padded to whole tiles with zero weights, so nothing in
// either part is masked but the last stores.
// Bound: one workgroup's chain of dependent products, LDS reads and
// activations.  The lane-per-entry form above reads both operands of every
// product from LDS one float at a time and passes eight barriers per epoch of
// a three-layer network: 11.6 us for 33-16-16-3 on 120 rows, here 3.9.
using mlph::DeepTilePlan;
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// HT: unit tiles of the widest hidden layer; LC: layers; ACT: 0 sigma, 1 tanh;
// RAG: a hidden layer has fewer tiles than HT, and the loops over its tiles stop
// there (uniform branches; without them the padding of narrow layers beside a
// wide one costs more than the matrix cores gain: 4-8-4-48-1 on 3 rows 9.7 us an
// epoch, with them 6.0, in the form above 7.2).
template <int HT, int ACT, int LC, bool RAG>
__global__ __launch_bounds__(64 * mlph::kDeepTileWaves) void k_deep_tiled(
    DeepTilePlan p, const float *__restrict__ X, const float *__restrict__ T, float *__restrict__ theta,
    float *__restrict__ comp, float lr, int epochs, float *__restrict__ loss_hist) {
  extern __shared__ float4 smem4[];
  float *sm = reinterpret_cast<float *>(smem4);
  const int NT = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int n = p.n, P = p.P, K = p.w[LC], NW = p.NW, NPT = p.NPT;
  const bool compensated = comp != nullptr;
  constexpr int SH = 16 * HT + 4, ST = 20;   // row strides of hidden-layer and output arrays

  // ---- rows, targets and parameters; everything else (padding) is zero
  for (int i = tid; i < p.total; i += NT) sm[i] = 0.0f;
  __syncthreads();
  const int D = p.w[0], SX = p.sx, IT0 = p.it0;
  for (int i = tid; i < n * D; i += NT) {
    const int r = i / D, c = i - r * D;
    sm[p.aoff[0] + r * SX + c] = X[i];
  }
  for (int i = tid; i < n * K; i += NT) {
    const int r = i / K, k = i - r * K;
    sm[p.toff + r * ST + k] = T[i];
  }
  // LDS place of packed parameter q (weights, or compensation terms cdelta on)
  auto place = [&](int q) {
    int l = 0;
    while (l + 1 < LC && q >= p.poff[l + 1]) ++l;
    const int wi = p.w[l], o = q - p.poff[l], nw = wi * p.w[l + 1];
    return o < nw ? p.woff[l] + o / wi * (l ? SH : SX) + o % wi : p.boff[l] + (o - nw);
  };
  for (int q = tid; q < P; q += NT) {
    const int at = place(q);
    sm[at] = theta[q];
    if (compensated) sm[at + p.cdelta] = comp[q];
  }
  __syncthreads();

  // unit tiles of layer l's outputs, and of its inputs above the first layer
  auto tiles_out = [&](int l) { return l == LC - 1 ? 1 : RAG ? (p.w[l + 1] + 15) >> 4 : HT; };
  auto tiles_in = [&](int l) { return RAG ? (p.w[l] + 15) >> 4 : HT; };

  const float dscale = 2.0f / ((float)n * (float)K);
  const float inv_nk = 1.0f / ((float)n * (float)K);

  for (int e = 0; e < epochs; ++e) {
    // ======================= rows
    float sq = 0.0f;
    for (int rt = wave; rt < NPT; rt += NW) {
      const int row = rt * 16 + l16;
      f32x4_t a[LC][HT];   // outputs of layer l (the top layer's in tile 0)
#pragma unroll
      for (int l = 0; l < LC; ++l) {
        constexpr int kTop = LC - 1;
        const int OT = tiles_out(l);
        const int s0 = l ? SH : SX;
        const float *W = sm + p.woff[l] + l16 * s0 + 4 * lg;
        f32x4_t z[HT];
#pragma unroll
        for (int t = 0; t < HT; ++t)
          if (t < OT) z[t] = *reinterpret_cast<const f32x4_t *>(sm + p.boff[l] + 16 * t + 4 * lg);
        auto tile = [&](int it, f32x4_t in) {   // inputs 16 it .. of this row
#pragma unroll
          for (int t = 0; t < HT; ++t) {
            if (t < OT) {
              const f32x4_t wv = *reinterpret_cast<const f32x4_t *>(W + t * 16 * s0 + 16 * it);
#pragma unroll
              for (int s = 0; s < 4; ++s) z[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[s], in[s], z[t], 0, 0, 0);
            }
          }
        };
        if (l == 0) {
          const float *x = sm + p.aoff[0] + row * SX + 4 * lg;
          for (int it = 0; it < IT0; ++it) tile(it, *reinterpret_cast<const f32x4_t *>(x + 16 * it));
        } else {
#pragma unroll
          for (int it = 0; it < HT; ++it)
            if (it < tiles_in(l)) tile(it, a[l ? l - 1 : 0][it]);
        }
#pragma unroll
        for (int t = 0; t < HT; ++t) {
          if (t < OT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) a[l][t][i] = (l < kTop && ACT == 1) ? tanhf(z[t][i]) : sigmoid(z[t][i]);
            if (l < kTop)
              *reinterpret_cast<f32x4_t *>(sm + p.aoff[l + 1 < LC ? l + 1 : 0] + row * SH + 16 * t + 4 * lg) = a[l][t];
          }
        }
      }
      // error and the top layer's delta
      f32x4_t d[HT];
      {
        const f32x4_t tv = *reinterpret_cast<const f32x4_t *>(sm + p.toff + row * ST + 4 * lg);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float y = a[LC - 1][0][i], err = row < n && 4 * lg + i < K ? y - tv[i] : 0.0f;
          sq = fmaf(err, err, sq);
          d[0][i] = (dscale * err) * (y * (1.0f - y));
        }
        *reinterpret_cast<f32x4_t *>(sm + p.doff[LC - 1] + row * ST + 4 * lg) = d[0];
      }
      // the deltas below, through the pre-update weights
#pragma unroll
      for (int l = LC - 1; l > 0; --l) {
        const int OT = tiles_out(l);
        f32x4_t dn[HT];
        const float *W = sm + p.woff[l] + 4 * lg * SH + l16;
#pragma unroll
        for (int it = 0; it < HT; ++it) {
          if (it >= tiles_in(l)) break;
          f32x4_t b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int t = 0; t < HT; ++t)
            if (t < OT) {
#pragma unroll
              for (int s = 0; s < 4; ++s)
                b = __builtin_amdgcn_mfma_f32_16x16x4f32(W[(16 * t + s) * SH + 16 * it], d[t][s], b, 0, 0, 0);
            }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float av = a[l - 1][it][i];
            b[i] *= ACT == 1 ? 1.0f - av * av : av * (1.0f - av);
          }
          *reinterpret_cast<f32x4_t *>(sm + p.doff[l - 1] + row * SH + 16 * it + 4 * lg) = b;
          dn[it] = b;
        }
#pragma unroll
        for (int t = 0; t < HT; ++t) d[t] = dn[t];
      }
    }
    sq = wave_sum(sq);
    if (lane == 0) sm[p.red + wave] = sq;
    __syncthreads();

    // ======================= weights: tile j (of layer l, units 16 ot, inputs 16 it)
    if (loss_hist && wave == NW - 1) {
      // (the last wave owns the fewest tiles)
      float s = lane < min(NW, NPT) ? sm[p.red + lane] : 0.0f;
      s = wave_sum(s);
      if (lane == 0) loss_hist[e] = s * inv_nk;
    }
    for (int j = wave; j < p.tiles; j += NW) {
      int l, it, ot;
      if (j < HT * IT0) {
        l = 0;
        it = j / HT;
        ot = j - it * HT;
      } else {
        const int k = j - HT * IT0;
        l = 1 + min(k / (HT * HT), LC - 2);
        const int r = k - (l - 1) * HT * HT;
        it = l == LC - 1 ? r : r / HT;
        ot = l == LC - 1 ? 0 : r - it * HT;
      }
      const int sa = l ? SH : SX, sd = l == LC - 1 ? ST : SH, wi = p.w[l], wo = p.w[l + 1];
      if (RAG && (16 * it >= wi || 16 * ot >= wo)) continue;   // only padding
      const float *Dp = sm + p.doff[l] + lg * sd + 16 * ot + l16;
      const float *Ap = sm + p.aoff[l] + lg * sa + 16 * it + l16;
      // row tiles in pairs whose chains overlap, each from zero and added to
      // the totals: chains over all rows err like a rounding per row (120 rows
      // of 33-16-16-3, rms error of a step's gradients 10.0e-9 of the largest,
      // so 6.8e-9, for 3.95 us an epoch instead of 3.73); a row tile past the
      // end is not read (NPT odd)
      f32x4_t g0 = {0.f, 0.f, 0.f, 0.f}, g1 = {0.f, 0.f, 0.f, 0.f};
      float gb = 0.0f;
      int rt = 0;
      for (; rt + 2 <= NPT; rt += 2) {
        float dv[8], av[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          dv[s] = Dp[(16 * rt + 4 * s) * sd];
          av[s] = Ap[(16 * rt + 4 * s) * sa];
        }
        f32x4_t p0 = {0.f, 0.f, 0.f, 0.f}, p1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          p0 = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[s], av[s], p0, 0, 0, 0);
          p1 = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[4 + s], av[4 + s], p1, 0, 0, 0);
          gb += dv[s] + dv[4 + s];
        }
        g0 += p0;
        g1 += p1;
      }
      if (rt < NPT) {
        f32x4_t p0 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float dv = Dp[(16 * rt + 4 * s) * sd];
          p0 = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, Ap[(16 * rt + 4 * s) * sa], p0, 0, 0, 0);
          gb += dv;
        }
        g0 += p0;
      }
      const int i0 = 16 * it + l16;
      float *Wt = sm + p.woff[l] + (16 * ot + 4 * lg) * sa + i0;
      float wv[4], cv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        wv[i] = Wt[i * sa];
        cv[i] = Wt[i * sa + p.cdelta];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        gd_update(wv[i], cv[i], lr, g0[i] + g1[i], compensated);
        if (i0 < wi && 16 * ot + 4 * lg + i < wo) {
          Wt[i * sa] = wv[i];
          Wt[i * sa + p.cdelta] = cv[i];
        }
      }
      if (it == 0) {   // the tile that also sums its units' bias gradients
        gb = sum_rows(gb);
        const int o = 16 * ot + l16;
        if (lg == 0 && o < wo) {
          float *bp = sm + p.boff[l] + o;
          float b = *bp, c = bp[p.cdelta];
          gd_update(b, c, lr, gb, compensated);
          *bp = b;
          bp[p.cdelta] = c;
        }
      }
    }
    __syncthreads();
  }

  for (int q = tid; q < P; q += NT) {
    const int at = place(q);
    theta[q] = sm[at];
    if (compensated) comp[q] = sm[at + p.cdelta];
  }
}

}  // namespace mlpk

namespace mlph {

bool deep_tile_plan(int L, const int32_t *widths, int64_t n, size_t lds_max, DeepTilePlan *p) {
  if (L < 2 || L > kDeepTileLayers || n < 1 || n > (1 << 20) || widths[L] > 16) return false;
  DeepTilePlan q{};
  const int64_t cap = (int64_t)(lds_max / sizeof(float));
  int64_t o = 0;
  q.n = (int)n;
  q.NPT = (int)((n + 15) / 16);
  q.ht = 1;
  for (int l = 0; l <= L; ++l) {
    if (widths[l] < 1 || widths[l] > kDeepMaxWidth || (l > 0 && widths[l] > kDeepTileWidth)) return false;
    q.w[l] = widths[l];
    if (l > 0 && l < L) q.ht = std::max(q.ht, (widths[l] + 15) / 16);
  }
  if (q.ht == 3) q.ht = 4;   // the kernel instances
  q.it0 = (widths[0] + 15) / 16;
  q.sx = 16 * q.it0 + 4;
  const int sh = 16 * q.ht + 4, st = 20;
  const int64_t rows = 16 * (int64_t)q.NPT;
  auto take = [&](int64_t floats) {   // an array of this many floats (a multiple of 4)
    const int64_t at = o;
    o = std::min(o + floats, cap + 1);
    return (int)at;
  };
  int64_t P = 0;
  const int64_t w0 = o;
  for (int l = 0; l < L; ++l) {
    q.poff[l] = (int)P;
    P += (int64_t)widths[l + 1] * widths[l] + widths[l + 1];
    const int units = l == L - 1 ? 16 : 16 * q.ht;
    q.woff[l] = take((int64_t)units * (l ? sh : q.sx));
    q.boff[l] = take(units);
  }
  q.P = (int)P;
  q.cdelta = (int)(o - w0);   // compensation terms lie like the weights
  take(o - w0);
  for (int l = 0; l < L; ++l) {
    q.aoff[l] = take(rows * (l ? sh : q.sx));
    q.doff[l] = take(rows * (l == L - 1 ? st : sh));
  }
  q.toff = take(rows * st);
  q.red = take(kDeepTileWaves);
  if (o > cap) return false;
  q.tiles = q.ht * q.it0 + (L - 2) * q.ht * q.ht + q.ht;
  q.NW = std::min(kDeepTileWaves, std::max(4, std::max(q.NPT, q.tiles)));
  q.total = (int)o;
  *p = q;
  return true;
}

template <int ACT, int LC>
static const void *deep_tiled_kernel(int ht, bool ragged) {
  using namespace mlpk;
  if (ht == 4) return ragged ? (const void *)k_deep_tiled<4, ACT, LC, true> : (const void *)k_deep_tiled<4, ACT, LC, false>;
  return ht == 1 ? (const void *)k_deep_tiled<1, ACT, LC, false> : (const void *)k_deep_tiled<2, ACT, LC, false>;
}

hipError_t launch_deep_train_tiled(const DeepTilePlan &p, int n_layers, int act, const float *X, const float *T,
                                   float *theta, float *comp, float lr, int epochs, float *loss_hist, hipStream_t s) {
  // the branches pay where at most 0.7 of the padded tiles are real (an epoch on
  // 2 rows with and without: 48-50-48-32-1, 0.67, 10.9 / 11.1 us; 16-33-64-4, 0.79,
  // 8.0 / 7.7; 16-33-50-50-2, 0.88, 11.7 / 9.8)
  int real = 0;
  for (int l = 0; l < n_layers; ++l) real += (p.w[l] + 15) / 16 * ((p.w[l + 1] + 15) / 16);
  const bool ragged = 10 * real <= 7 * p.tiles;
  const void *kern = n_layers == 2   ? (act ? deep_tiled_kernel<1, 2>(p.ht, ragged) : deep_tiled_kernel<0, 2>(p.ht, ragged))
                     : n_layers == 3 ? (act ? deep_tiled_kernel<1, 3>(p.ht, ragged) : deep_tiled_kernel<0, 3>(p.ht, ragged))
                                     : (act ? deep_tiled_kernel<1, 4>(p.ht, ragged) : deep_tiled_kernel<0, 4>(p.ht, ragged));
  const size_t lds = (size_t)p.total * sizeof(float);
  hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  DeepTilePlan plan = p;
  void *args[] = {&plan, &X, &T, &theta, &comp, &lr, &epochs, &loss_hist};
  e = hipLaunchKernel(kern, dim3(1), dim3(64 * p.NW), args, lds, s);
  return e == hipSuccess ? hipGetLastError() : e;
}

bool deep_plan(int L, const int32_t *widths, int64_t n, size_t lds_max, DeepPlan *p) {
  if (L < 1 || L > kDeepMaxLayers || n < 1 || n > (1 << 20)) return false;
  for (int l = 0; l <= L; ++l)
    if (widths[l] < 1 || widths[l] > kDeepMaxWidth) return false;
  DeepPlan q{};
  q.L = L;
  q.n = (int)n;
  int64_t P = 0;
  for (int l = 0; l <= L; ++l) {
    q.w[l] = widths[l];
    q.sa[l] = (widths[l] + 1) | 1;   // room for the column of ones
    q.poff[l] = (int)P;
    if (l < L) P += (int64_t)widths[l + 1] * widths[l] + widths[l + 1];
  }
  const int64_t cap = (int64_t)(lds_max / sizeof(float));
  if (P > cap) return false;
  q.P = (int)P;
  int64_t o = 0;
  for (int l = 0; l <= L; ++l) {
    q.aoff[l] = (int)std::min<int64_t>(o, cap);
    o += n * q.sa[l];
    if (o > cap) return false;
  }
  q.toff = (int)o;
  o += n * q.sa[L];
  int sd = 1;
  for (int l = 1; l <= L; ++l) sd = std::max(sd, q.sa[l]);
  q.sd = sd;
  q.d0 = (int)std::min<int64_t>(o, cap);
  o += n * sd;
  q.d1 = (int)std::min<int64_t>(o, cap);
  o += n * sd;
  q.th = (int)std::min<int64_t>(o, cap);
  o += P;
  q.cp = (int)std::min<int64_t>(o, cap);
  o += P;
  q.red = (int)std::min<int64_t>(o, cap);
  o += kDeepThreads / 64;   // one slot per wave
  if (o > cap) return false;
  q.gr = (int)o;
  // the most row segments (8, 4, 2 or 1, each of at least 8 rows) that fit;
  // a segment's length is a multiple of 8 rows (the unroll of its sums) and
  // the last one takes what is left
  for (int rs = 8; rs >= 1; rs >>= 1) {
    const int64_t seg = ((n + rs - 1) / rs + 7) / 8 * 8;
    if (rs > 1 && (n + rs - 1) / rs < 8) continue;
    if (o + rs * P <= cap) {
      q.RS = rs;
      q.seg = (int)seg;
      q.total = (int)(o + rs * P);
      *p = q;
      return true;
    }
  }
  return false;
}

hipError_t launch_deep_train(const DeepPlan &p, int act, const float *X, const float *T, float *theta,
                             float *comp, float lr, int epochs, float *loss_hist, hipStream_t s) {
  const size_t lds = (size_t)p.total * sizeof(float);
  const void *kern = act == 1 ? (const void *)mlpk::k_deep_train<1> : (const void *)mlpk::k_deep_train<0>;
  hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  if (act == 1)
    hipLaunchKernelGGL(mlpk::k_deep_train<1>, dim3(1), dim3(kDeepThreads), lds, s, p, X, T, theta, comp, lr,
                       epochs, loss_hist);
  else
    hipLaunchKernelGGL(mlpk::k_deep_train<0>, dim3(1), dim3(kDeepThreads), lds, s, p, X, T, theta, comp, lr,
                       epochs, loss_hist);
  return hipGetLastError();
}

}  // namespace mlph
