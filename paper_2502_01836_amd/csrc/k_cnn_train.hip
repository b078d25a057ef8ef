// CNN filter training on FP32 matrix cores (v_mfma_f32_16x16x4_f32), for up to
// 96 channels: one work-group of eight wavefronts per filter, E examples of a
// mini-batch at a time.
//
// The second layer and both of its gradients are matrix products:
//   forward   z2[o][p]    = sum over (t, c) W2[o][c][t] h1[c][p + t - 1]
//   weights   dW2[o][c][t] = sum over p     d2[o][p]    h1[c][p + t - 1]
//   inputs    d1[c][x]    = sum over (t, o) W2[o][c][t] d2[o][x - t + 1]
// with h1 and d2 = dL/dz2 in LDS as [channel][position + 1], zero at both ends,
// so a tap is an offset into a row.  Wavefront w holds channel tile w mod MT
// (16 output channels forward, the same 16 input channels backward) of W2 in
// registers as the A operand and takes every ng-th of the E ceil(m / 16)
// column tiles; its pre-activations stay in registers until the prediction is
// known, then become d2.  The weight gradient's tiles (output x input channel
// tile, three taps) are dealt to the wavefronts, which accumulate theirs in
// registers over the whole mini-batch; with fewer than eight such tiles they
// share the positions of one.  Everything else (biases, readout, first layer)
// is accumulated per lane over the lane's columns.  Sums across lanes and
// wavefronts run in a fixed order once per mini-batch, then every weight is
// updated in place: no gradient buffer, no atomics.
//
// Row stride of h1 and d2: 20 or 44 mod 64 words, so that the 16 channels x 4
// positions of a weight-gradient operand hit 64 banks.
//
// 128 filters of 32 channels x 96 positions, batch 32: 5.29 ms (the plain
// kernel: one output per thread, operands re-read from LDS and global memory)
// -> 215 us (35 TFLOP/s), error of the losses against 64 bits 2.0e-7 -> 0.9e-7.
// Bound by the four barriers of a step and the LDS reads between them: one
// work-group per filter leaves half the CUs idle at 128 filters.
#include <algorithm>

#include "device_util.h"
#include "kernels.h"

namespace leafi {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kCtWaves = 8;
constexpr int kCtThreads = kWave * kCtWaves;
constexpr int kCtTiles = 6;     // column tiles of a wavefront
constexpr int kCtExamples = 4;  // most examples at a time

struct CtShape {
  int m, C, nt, R, E;  // positions, channels, column tiles of an example, row stride, examples at a time
};

__host__ __device__ inline int ct_ng(int mt) { return kCtWaves / mt; }
// Work-groups' parts of a weight-gradient tile's positions.
__host__ __device__ constexpr int ct_split(int mt) { return mt * mt >= kCtWaves ? 1 : kCtWaves / (mt * mt); }
__host__ __device__ constexpr int ct_pairs(int mt) { return mt * mt >= kCtWaves ? (mt * mt + kCtWaves - 1) / kCtWaves : 1; }

struct CtLds {
  float *xp;    // [E][R] padded examples
  float *h1;    // [E][16 MT][R]
  float *d2;    // [E][16 MT][R]; after a batch the parts of split weight-gradient tiles
  float4 *w1s;  // [C] first-layer taps and bias
  float *red;   // [waves][kCtExamples]
  float *sred;  // [ng][16 MT][6] per-channel sums of each column group
  float *b3;    // [4] output bias; validation error; stop
};
__host__ __device__ inline int ct_d2_floats(const CtShape &s, int mt) {
  const int act = s.E * 16 * mt * s.R, parts = (ct_split(mt) - 1) * mt * mt * 12 * kWave;
  return act > parts ? act : parts;
}
__host__ __device__ inline size_t ct_lds_floats(const CtShape &s, int mt) {
  return (static_cast<size_t>(s.E) * s.R + 3) / 4 * 4 + static_cast<size_t>(s.E) * 16 * mt * s.R + ct_d2_floats(s, mt) +
         4 * static_cast<size_t>(s.C) + kCtWaves * kCtExamples + static_cast<size_t>(ct_ng(mt)) * 16 * mt * 6 + 4;
}
__device__ inline CtLds ct_carve(float *base, const CtShape &s, int mt) {
  CtLds l;
  l.xp = base;
  l.h1 = l.xp + (s.E * s.R + 3) / 4 * 4;
  l.d2 = l.h1 + s.E * 16 * mt * s.R;
  l.w1s = reinterpret_cast<float4 *>(l.d2 + ct_d2_floats(s, mt));
  l.red = reinterpret_cast<float *>(l.w1s + s.C);
  l.sred = l.red + kCtWaves * kCtExamples;
  l.b3 = l.sred + ct_ng(mt) * 16 * mt * 6;
  return l;
}

// Sum over the 16 lanes of a quarter (fixed butterfly).
__device__ __forceinline__ float quarter_sum(float v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// One mini-batch of nb examples (row(e), target(e)) through the filter whose
// packed weights are wf (b3 in l.b3[0]): the sum of squared errors, and with
// Update the SGD step.  Every thread of the work-group calls it; LDS rows are
// zero outside the positions and channels in use.
template <int MT, bool Update, typename Row, typename Target>
__device__ float ct_batch(float *wf, int nb, float lr, const CtShape &s, const CtLds &l, Row row, Target target) {
  constexpr int KC = 4 * MT;  // 4-channel steps
  constexpr int SP = ct_split(MT), GP = ct_pairs(MT);
  const int m = s.m, C = s.C, R = s.R, nt = s.nt, E = s.E;
  int tid = threadIdx.x;
  int lane = tid & (kWave - 1), col = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int tile = wave % MT, pg = wave / MT, ng = ct_ng(MT);
  const bool act = pg < ng;
  float *W2 = wf + 4 * C, *b2p = W2 + 3 * C * C, *w3p = b2p + C;
  const float inv_m = 1.0f / static_cast<float>(m);
  for (int c = tid; c < C; c += kCtThreads)
    l.w1s[c] = make_float4(wf[3 * c], wf[3 * c + 1], wf[3 * c + 2], wf[3 * C + c]);
  // A operands: forward row o = 16 tile + col, channel 4 ks + q; backward row
  // c = 16 tile + col, output channel 4 ks + q
  float FA[3][KC], HA[3][Update ? KC : 1];
#pragma unroll
  for (int ks = 0; ks < KC; ++ks) {
    const int r = 16 * tile + col, k = 4 * ks + q;
    const bool in = r < C && k < C;
    const float *pf = W2 + (in ? (r * C + k) * 3 : 0), *ph = W2 + (in ? (k * C + r) * 3 : 0);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const float vf = pf[t];
      FA[t][ks] = in ? vf : 0.0f;
      if constexpr (Update) {
        const float vh = ph[t];
        HA[t][ks] = in ? vh : 0.0f;
      }
    }
  }
  float b2[4], w3[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int j = 16 * tile + 4 * q + r;
    b2[r] = j < C ? b2p[j] : 0.0f;
    w3[r] = j < C ? w3p[j] : 0.0f;
  }
  floatx4 G[GP][3];
  float gb2[4], gw3[4], gb1[4], gw1[4][3], gb3 = 0.0f, sse = 0.0f;
#pragma unroll
  for (int i = 0; i < GP; ++i)
#pragma unroll
    for (int t = 0; t < 3; ++t) G[i][t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    gb2[r] = gw3[r] = gb1[r] = 0.0f;
    gw1[r][0] = gw1[r][1] = gw1[r][2] = 0.0f;
  }
  for (int e0 = 0; e0 < nb; e0 += E) {
    const int ne = nb - e0 < E ? nb - e0 : E;
    // opaque, so that the unrolled tiles' addresses are derived again in every
    // step instead of being kept in registers (and spilled) across the steps
    asm volatile("" : "+v"(tid));
    lane = tid & (kWave - 1);
    col = lane & 15;
    q = lane >> 4;
    // rows past ne are stale: no column tile reads them
    for (int i = tid; i < ne * m; i += kCtThreads) {
      const int e = i / m, p = i - e * m;
      l.xp[e * R + p + 1] = row(e0 + e)[p];
    }
    __syncthreads();  // rows and first-layer weights staged; the previous step's readers are done
    for (int i = tid; i < ne * C * m; i += kCtThreads) {
      const int ec = i / m, p = i - ec * m, e = ec / C, c = ec - e * C;
      const float4 u = l.w1s[c];
      const float *xp = l.xp + e * R + p;
      float z = u.w;
      z = fmaf(u.x, xp[0], z);
      z = fmaf(u.y, xp[1], z);
      z = fmaf(u.z, xp[2], z);
      l.h1[(e * 16 * MT + c) * R + p + 1] = fmaxf(z, 0.0f);
    }
    __syncthreads();
    // forward
    floatx4 Z[kCtTiles];
    float pe[kCtExamples];
#pragma unroll
    for (int e = 0; e < kCtExamples; ++e) pe[e] = 0.0f;
#pragma unroll
    for (int i = 0; i < kCtTiles; ++i) {
      const int ct = pg + ng * i;
      Z[i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      if (act && ct < ne * nt) {  // uniform
        const int e = ct / nt, p = 16 * (ct - e * nt) + col;
        const float *hb = l.h1 + (e * 16 * MT + q) * R + p;
#pragma unroll
        for (int ks = 0; ks < KC; ++ks)
#pragma unroll
          for (int t = 0; t < 3; ++t)
            Z[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(FA[t][ks], hb[4 * ks * R + t], Z[i], 0, 0, 0);
        float v = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          Z[i][r] = p < m ? Z[i][r] + b2[r] : 0.0f;
          v = fmaf(w3[r], fmaxf(Z[i][r], 0.0f), v);
        }
#pragma unroll
        for (int x = 0; x < kCtExamples; ++x) pe[x] += x == e ? v : 0.0f;
      }
    }
#pragma unroll
    for (int e = 0; e < kCtExamples; ++e)
      if (e < ne) {  // uniform
        const float v = wave_sum(pe[e]);
        if (lane == 0) l.red[wave * kCtExamples + e] = v;
      }
    __syncthreads();
    float g[kCtExamples];
#pragma unroll
    for (int e = 0; e < kCtExamples; ++e) {
      g[e] = 0.0f;
      if (e < ne) {
        float v = 0.0f;
        for (int w = 0; w < kCtWaves; ++w) v += l.red[w * kCtExamples + e];
        const float err = fmaf(v, inv_m, l.b3[0]) - target(e0 + e);
        sse = fmaf(err, err, sse);
        g[e] = 2.0f * err / static_cast<float>(nb);
        gb3 += g[e];
      }
    }
    if constexpr (Update) {
      // dL/dz2 into LDS; the readout's and the second bias's sums
#pragma unroll
      for (int i = 0; i < kCtTiles; ++i) {
        const int ct = pg + ng * i;
        if (act && ct < ne * nt) {
          const int e = ct / nt, p = 16 * (ct - e * nt) + col;
          float ge = 0.0f;
#pragma unroll
          for (int x = 0; x < kCtExamples; ++x) ge = x == e ? g[x] : ge;
          const float gm = ge * inv_m;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float z = Z[i][r], d = z > 0.0f ? gm * w3[r] : 0.0f;
            gb2[r] += d;
            gw3[r] = fmaf(gm, fmaxf(z, 0.0f), gw3[r]);
            if (p < m) l.d2[(e * 16 * MT + 16 * tile + 4 * q + r) * R + p + 1] = d;
          }
        }
      }
      __syncthreads();
      // weight gradient
#pragma unroll
      for (int i = 0; i < GP; ++i) {
        const int pair = SP > 1 ? wave % (MT * MT) : wave + kCtWaves * i;
        const int part = SP > 1 ? wave / (MT * MT) : 0;
        if (pair < MT * MT && part < SP) {  // uniform
          const int ot = pair / MT, ic = pair - ot * MT;
          for (int e = 0; e < ne; ++e) {
            const float *da = l.d2 + (e * 16 * MT + 16 * ot + col) * R + q + 1;
            const float *hb = l.h1 + (e * 16 * MT + 16 * ic + col) * R + q;
#pragma unroll 4
            for (int ks = part; ks < m / 4; ks += SP) {
              const float a = da[4 * ks];
#pragma unroll
              for (int t = 0; t < 3; ++t)
                G[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, hb[4 * ks + t], G[i][t], 0, 0, 0);
            }
          }
        }
      }
      // input gradient, and from it the first layer's sums
#pragma unroll
      for (int i = 0; i < kCtTiles; ++i) {
        const int ct = pg + ng * i;
        if (act && ct < ne * nt) {
          const int e = ct / nt, x = 16 * (ct - e * nt) + col;
          const float *db = l.d2 + (e * 16 * MT + q) * R + x;
          floatx4 D = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int ks = 0; ks < KC; ++ks)
#pragma unroll
            for (int t = 0; t < 3; ++t)
              D = __builtin_amdgcn_mfma_f32_16x16x4f32(HA[t][ks], db[4 * ks * R + 2 - t], D, 0, 0, 0);
          const float *xr = l.xp + e * R + x;
          const float x0 = xr[0], x1 = xr[1], x2 = xr[2];
          const float *hr = l.h1 + (e * 16 * MT + 16 * tile + 4 * q) * R + x + 1;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float d = x < m && hr[r * R] > 0.0f ? D[r] : 0.0f;
            gb1[r] += d;
            gw1[r][0] = fmaf(d, x < m ? x0 : 0.0f, gw1[r][0]);
            gw1[r][1] = fmaf(d, x < m ? x1 : 0.0f, gw1[r][1]);
            gw1[r][2] = fmaf(d, x < m ? x2 : 0.0f, gw1[r][2]);
          }
        }
      }
    }
    __syncthreads();
  }
  if constexpr (Update) {
    // per-channel sums of the wavefront's columns, then over the column groups
    if (act) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v[6] = {gb2[r], gw3[r], gb1[r], gw1[r][0], gw1[r][1], gw1[r][2]};
        float *o = l.sred + (pg * 16 * MT + 16 * tile + 4 * q + r) * 6;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          v[i] = quarter_sum(v[i]);
          if (col == 0) o[i] = v[i];
        }
      }
    }
    if constexpr (SP > 1) {
      const int pair = wave % (MT * MT), part = wave / (MT * MT);
      if (part > 0 && part < SP) {
        float *o = l.d2 + ((part - 1) * MT * MT + pair) * 12 * kWave + lane;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[(4 * t + r) * kWave] = G[0][t][r];
      }
    }
    __syncthreads();
    if constexpr (SP > 1) {
      const int pair = wave % (MT * MT), part = wave / (MT * MT);
      if (part == 0)
        for (int x = 1; x < SP; ++x) {
          const float *o = l.d2 + ((x - 1) * MT * MT + pair) * 12 * kWave + lane;
#pragma unroll
          for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) G[0][t][r] += o[(4 * t + r) * kWave];
        }
    }
#pragma unroll
    for (int i = 0; i < GP; ++i) {
      const int pair = SP > 1 ? wave % (MT * MT) : wave + kCtWaves * i;
      const int part = SP > 1 ? wave / (MT * MT) : 0;
      if (pair < MT * MT && part == 0) {
        const int ot = pair / MT, ic = pair - ot * MT;
        const int c = 16 * ic + col;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int o = 16 * ot + 4 * q + r;
          if (o < C && c < C) {
            float *p = W2 + (o * C + c) * 3;
#pragma unroll
            for (int t = 0; t < 3; ++t) p[t] = fmaf(-lr, G[i][t][r], p[t]);
          }
        }
      }
    }
    for (int c = tid; c < C; c += kCtThreads) {
      float v[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
      for (int g = 0; g < ng; ++g)
#pragma unroll
        for (int i = 0; i < 6; ++i) v[i] += l.sred[(g * 16 * MT + c) * 6 + i];
      b2p[c] = fmaf(-lr, v[0], b2p[c]);
      w3p[c] = fmaf(-lr, v[1], w3p[c]);
      wf[3 * C + c] = fmaf(-lr, v[2], wf[3 * C + c]);
#pragma unroll
      for (int t = 0; t < 3; ++t) wf[3 * c + t] = fmaf(-lr, v[3 + t], wf[3 * c + t]);
    }
    if (tid == 0) l.b3[0] = fmaf(-lr, gb3, l.b3[0]);
    // the parts in d2 are consumed: its rows are zero outside the positions again
    if constexpr (SP > 1) {
      __syncthreads();
      const int n = s.E * 16 * MT * R, parts = (SP - 1) * MT * MT * 12 * kWave;
      for (int i = tid; i < (n < parts ? n : parts); i += kCtThreads) l.d2[i] = 0.0f;
    }
    __syncthreads();  // the updated weights are read by every wavefront of the next batch
  }
  return sse;
}

__device__ inline void ct_clear(float *lds, const CtShape &s, int mt) {
  const int n = static_cast<int>(ct_lds_floats(s, mt));
  for (int i = threadIdx.x; i < n; i += kCtThreads) lds[i] = 0.0f;
}

template <int MT>
__global__ void __launch_bounds__(kCtThreads, 2) k_cnn_sgd_step_mfma(float *w, CtShape s, const float *x,
                                                                     const float *y, int batch, float lr,
                                                                     float *loss) {
  extern __shared__ __align__(16) float lds[];
  const CtLds l = ct_carve(lds, s, MT);
  const int f = blockIdx.x;
  const int64_t P = 3LL * s.C * s.C + 6LL * s.C + 1;
  float *wf = w + f * P;
  ct_clear(lds, s, MT);
  __syncthreads();
  if (threadIdx.x == 0) l.b3[0] = wf[P - 1];
  const float *xf = x + static_cast<int64_t>(f) * batch * s.m, *yf = y + static_cast<int64_t>(f) * batch;
  __syncthreads();
  const float sse = ct_batch<MT, true>(
      wf, batch, lr, s, l, [=](int e) { return xf + static_cast<int64_t>(e) * s.m; }, [=](int e) { return yf[e]; });
  if (threadIdx.x == 0) {
    wf[P - 1] = l.b3[0];
    loss[f] = sse / static_cast<float>(batch);
  }
}

// The whole SGD run of one filter per work-group, with k_cnn_train's schedule
// (shuffled epochs, validation after each, the learning rate divided by 10
// after `patience` epochs without a 1e-4 relative improvement, stop below
// lr_min, best-validation weights kept).
template <int MT>
__global__ void __launch_bounds__(kCtThreads, 2) k_cnn_train_mfma(TrainArgs a, CtShape s) {
  extern __shared__ __align__(16) float lds[];
  const CtLds l = ct_carve(lds, s, MT);
  int32_t *perm = reinterpret_cast<int32_t *>(l.b3 + 4);  // [n_train]
  const int m = a.m, f = blockIdx.x;
  const int64_t P = 3LL * s.C * s.C + 6LL * s.C + 1;
  float *wf = a.w + f * P, *wb = a.w_best + f * P;
  const int32_t *exq = a.ex_q + static_cast<int64_t>(f) * a.n_ex;
  const float *exy = a.ex_y + static_cast<int64_t>(f) * a.n_ex;
  const int n_val = a.n_ex - a.n_train;
  ct_clear(lds, s, MT);
  __syncthreads();
  // output bias starts at the mean training target
  if (threadIdx.x == 0) {
    double acc = 0.0;
    for (int e = 0; e < a.n_train; ++e) acc += exy[e];
    l.b3[0] = static_cast<float>(acc / (a.n_train > 0 ? a.n_train : 1));
    wf[P - 1] = l.b3[0];
  }
  for (int e = threadIdx.x; e < a.n_train; e += kCtThreads) perm[e] = e;
  __syncthreads();
  for (int64_t e = threadIdx.x; e < P; e += kCtThreads) wb[e] = wf[e];
  float best = __builtin_inff(), lr = a.lr0;
  int bad = 0, epoch = 0;
  for (; epoch < a.max_epochs; ++epoch) {
    if (threadIdx.x == 0) {  // Fisher-Yates shuffle with a counter-based generator
      for (int e = a.n_train - 1; e > 0; --e) {
        uint64_t r = mix64(a.seed ^ mix64((static_cast<uint64_t>(f) << 40) ^ (static_cast<uint64_t>(epoch) << 20) ^ e));
        int o = static_cast<int>(r % static_cast<uint64_t>(e + 1));
        int tmp = perm[e];
        perm[e] = perm[o];
        perm[o] = tmp;
      }
    }
    __syncthreads();
    for (int s0 = 0; s0 < a.n_train; s0 += a.batch) {
      const int nb = a.n_train - s0 < a.batch ? a.n_train - s0 : a.batch;
      ct_batch<MT, true>(
          wf, nb, lr, s, l, [=](int e) { return a.xq + static_cast<int64_t>(exq[perm[s0 + e]]) * m; },
          [=](int e) { return exy[perm[s0 + e]]; });
    }
    // validation error (forward passes only)
    float vm = 0.0f;
    if (n_val > 0)
      vm = ct_batch<MT, false>(
               wf, n_val, 0.0f, s, l, [=](int e) { return a.xq + static_cast<int64_t>(exq[a.n_train + e]) * m; },
               [=](int e) { return exy[a.n_train + e]; }) /
           n_val;
    if (threadIdx.x == 0) {
      wf[P - 1] = l.b3[0];
      if (a.val_trace) a.val_trace[static_cast<int64_t>(f) * a.max_epochs + epoch] = vm;
    }
    __syncthreads();
    const bool improved = vm < best * (1.0f - 1e-4f);
    if (improved) {
      best = vm;
      bad = 0;
      for (int64_t e = threadIdx.x; e < P; e += kCtThreads) wb[e] = wf[e];
    } else if (++bad >= a.patience) {
      lr *= 0.1f;
      bad = 0;
    }
    // every thread holds the same sums, so all of them agree on the end
    if ((lr < a.lr_min * (1.0f - 1e-3f)) || !(vm == vm)) {
      ++epoch;
      break;
    }
    __syncthreads();
  }
  __syncthreads();
  for (int64_t e = threadIdx.x; e < P; e += kCtThreads) wf[e] = wb[e];
  if (threadIdx.x == 0) {
    a.val_mse[f] = best;
    a.epochs_run[f] = epoch;
  }
}

// The largest number of examples at a time whose column tiles the wavefronts
// hold and whose activations fit in LDS beside `extra` bytes; E = 0: none.
CtShape ct_shape(int m, int C, size_t extra) {
  const int mt = (C + 15) / 16;
  CtShape s{m, C, (m + 15) / 16, 0, 0};
  s.R = 16 * s.nt + 2;
  while (s.R % 64 != 20 && s.R % 64 != 44) ++s.R;
  if (mt > 6) return s;
  for (int e = kCtExamples; e >= 1; e /= 2) {
    s.E = e;
    if (e * s.nt <= kCtTiles * ct_ng(mt) && ct_lds_floats(s, mt) * 4 + extra <= 160 * 1024) return s;
  }
  s.E = 0;
  return s;
}

template <int MT>
void ct_launch_step(const CtShape &s, float *w, int F, const float *x, const float *y, int batch, float lr, float *loss,
                    hipStream_t st) {
  const size_t lds = ct_lds_floats(s, MT) * 4;
  auto kern = k_cnn_sgd_step_mfma<MT>;
  allow_lds(reinterpret_cast<const void *>(kern), lds);
  hipLaunchKernelGGL(kern, dim3(F), dim3(kCtThreads), lds, st, w, s, x, y, batch, lr, loss);
  LAUNCH_OK("cnn_sgd_step_mfma");
}

template <int MT>
void ct_launch_train(const CtShape &s, const TrainArgs &a, hipStream_t st) {
  const size_t lds = ct_lds_floats(s, MT) * 4 + static_cast<size_t>(a.n_train) * 4;
  auto kern = k_cnn_train_mfma<MT>;
  allow_lds(reinterpret_cast<const void *>(kern), lds);
  hipLaunchKernelGGL(kern, dim3(a.F), dim3(kCtThreads), lds, st, a, s);
  LAUNCH_OK("cnn_train_mfma");
}

}  // namespace

bool launch_cnn_sgd_step_mfma(float *w, int F, int m, int C, const float *x, const float *y, int batch, float lr,
                              float *loss, hipStream_t st) {
  const CtShape s = ct_shape(m, C, 0);
  if (s.E == 0) return false;
  switch ((C + 15) / 16) {
    case 1: ct_launch_step<1>(s, w, F, x, y, batch, lr, loss, st); break;
    case 2: ct_launch_step<2>(s, w, F, x, y, batch, lr, loss, st); break;
    case 3: ct_launch_step<3>(s, w, F, x, y, batch, lr, loss, st); break;
    case 4: ct_launch_step<4>(s, w, F, x, y, batch, lr, loss, st); break;
    case 5: ct_launch_step<5>(s, w, F, x, y, batch, lr, loss, st); break;
    default: ct_launch_step<6>(s, w, F, x, y, batch, lr, loss, st); break;
  }
  return true;
}

bool launch_cnn_train_mfma(const TrainArgs &a, hipStream_t st) {
  const CtShape s = ct_shape(a.m, a.h, static_cast<size_t>(a.n_train) * 4);
  if (s.E == 0) return false;
  switch ((a.h + 15) / 16) {
    case 1: ct_launch_train<1>(s, a, st); break;
    case 2: ct_launch_train<2>(s, a, st); break;
    case 3: ct_launch_train<3>(s, a, st); break;
    case 4: ct_launch_train<4>(s, a, st); break;
    case 5: ct_launch_train<5>(s, a, st); break;
    default: ct_launch_train<6>(s, a, st); break;
  }
  return true;
}

}  // namespace leafi
