// CNN filter inference on the bf16 matrix cores at FP32 accuracy (three-part
// operands, split_bf16.h), for up to 128 channels and 256 positions.
//
// The second layer is a product of the weights (channels x (tap, channel))
// with the first layer's activations shifted by the tap.  Wavefront w holds
// the parts of 16 output channels (channel tile w mod mt) for every tap and
// input channel in registers, for as many rows as the work-group takes; the
// activations of one query lie in LDS as three bf16 planes [channel / 8]
// [position][8 channels] (position 0 and m + 1 zero), so the B operand of tap t
// is read at position p + t - 1 with no copy per tap, 16 positions of it
// consecutive (a position's channels side by side cost four more cycles per
// read in bank conflicts, a quarter of the kernel's time).  The planes are
// doubled: the wavefronts compute the next query's first layer between the
// products of the current one, with one barrier per query.
//
// 128 filters of 96 channels x 96 positions, 200 queries: 9.36 ms -> 623 us
// (221 TFLOP/s of FP32 products; error against 64 bits 2.6e-8 relative, as
// before) over the plain FP32 kernel, whose FMAs were fed from LDS by one
// work-group per filter (half the CUs).  Bound now by the matrix cores (half
// of the cycles) and the LDS reads of the B operand, three per six products.
#include <algorithm>

#include "kernels.h"
#include "split_bf16.h"

namespace leafi {

namespace {

constexpr int kConvMaxWaves = 12;

struct ConvArgs {
  const float *w;
  int F, m, C;
  const float *x;
  int64_t nq;            // dense form (plist null): out[q F + f]
  float *out;
  const int64_t *plist;  // listed form, as SplitArgs in the MLP inference
  const int32_t *pcnt;
  int64_t stride;
  int N;
  const int32_t *pair;
  const float *offsets;
  float *dfo;
  int mt, ng;            // 16-channel tiles, position groups
  int bufs;              // sets of planes: 2, or 1 where a work-group takes one query
};

// First-layer activation of a channel (its three taps, then its bias) at
// position p of the padded query (xp[p] is position p - 1).
__device__ __forceinline__ float conv_first(const float4 &u, const float *xp, int p) {
  float z = u.w;
  z = fmaf(u.x, xp[p], z);
  z = fmaf(u.y, xp[p + 1], z);
  z = fmaf(u.z, xp[p + 2], z);
  return fmaxf(z, 0.0f);
}

// The sum over channels o and positions p of w3[o] ReLU(z2[o][p]) in plain
// FP32, this thread's share; xp the padded query in LDS.
__device__ __forceinline__ float conv_plain(const float *__restrict__ wf, int m, int C, const float4 *w1s,
                                            const float *xp) {
  const float *W2 = wf + 4 * C, *b2 = W2 + 3 * C * C, *w3 = b2 + C;
  float sum = 0.0f;
  for (int e = threadIdx.x; e < C * m; e += blockDim.x) {
    const int o = e / m, p = e - o * m;
    float z = 0.0f;
    for (int c = 0; c < C; ++c)
      for (int t = 0; t < 3; ++t) {
        const int q = p + t - 1;
        if (q >= 0 && q < m) z = fmaf(W2[(o * C + c) * 3 + t], conv_first(w1s[c], xp, q), z);
      }
    sum = fmaf(w3[o], fmaxf(z + b2[o], 0.0f), sum);
  }
  return sum;
}

__host__ __device__ inline int conv_rows(int m) { return (m + 15) / 16 * 16 + 16; }  // positions per plane
__host__ __device__ inline int conv_xrow(int m) { return (m + 2 + 3) / 4 * 4; }
size_t conv_lds(int m, int C, int ks, int waves, int bufs) {
  return 3 * bufs * static_cast<size_t>(conv_rows(m)) * 32 * (ks / 3) * 2 + 3 * conv_xrow(m) * 4 + C * 16 +
         2 * waves * 4 + 32;
}

// KS: 32-wide steps of the product, three taps of KS / 3 channel blocks.
template <int KS>
__global__ void __launch_bounds__(KS <= 9 ? 768 : 512, KS <= 9 ? 3 : 2) k_cnn_infer_split(ConvArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int KB = KS / 3;            // 32-channel blocks
  constexpr int CP = 32 * KB;           // channels, padded
  const int f = blockIdx.x;
  const int64_t n = a.plist ? static_cast<int64_t>(a.pcnt[f]) : a.nq;
  if (static_cast<int64_t>(blockIdx.y) >= n) return;  // uniform
  const int m = a.m, C = a.C, T = blockDim.x;
  const int rows8 = conv_rows(m) * 8, plane = rows8 * (CP / 8), xrow = conv_xrow(m);
  uint16_t *planes = reinterpret_cast<uint16_t *>(smem);             // [bufs][3][CP / 8][positions][8]
  float *xs = reinterpret_cast<float *>(planes + 3 * a.bufs * plane);  // [3][xrow] padded queries
  float4 *w1s = reinterpret_cast<float4 *>(xs + 3 * xrow);           // [C] first-layer taps and bias
  float *red = reinterpret_cast<float *>(w1s + C);                   // [2][waves]
  int *bad = reinterpret_cast<int *>(red + 2 * (T / kWave));         // [4] queries, [1] weights
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 15, q = lane >> 4;
  const int tile = wave % a.mt, pg = wave / a.mt;
  const int64_t P = 3LL * C * C + 6LL * C + 1;
  const float *wf = a.w + f * P;
  const float *W2 = wf + 4 * C, *b2p = W2 + 3 * C * C, *w3p = b2p + C;
  // the planes' zero positions and channels stay zero; everything is cleared
  // once, so positions past m + 1 hold finite values too
  for (int e = tid; e < 3 * a.bufs * plane / 8; e += T)
    reinterpret_cast<uint4 *>(planes)[e] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < 5) bad[tid] = 0;
  for (int e = tid; e < 3 * xrow; e += T) xs[e] = 0.0f;
  // W2's parts: lane holds output channel 16 tile + col, step (tap t, block
  // kb): input channels 32 kb + 8 q .. + 8
  bf16x8 W[KS][3];
  float b2[4], w3[4];
  bool oddw = false;
  {
    const int o = 16 * tile + col;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      // the three taps of a channel are consecutive
      float raw[3][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int c = 32 * kb + 8 * q + e;
        const bool in = o < C && c < C;
        const float *p = W2 + (in ? (static_cast<uint32_t>(o) * C + c) * 3 : 0);
#pragma unroll
        for (int t = 0; t < 3; ++t) raw[t][e] = in ? p[t] : 0.0f;
      }
#pragma unroll
      for (int t = 0; t < 3; ++t) oddw |= split8(raw[t], W[3 * kb + t][0], W[3 * kb + t][1], W[3 * kb + t][2]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // the products' output rows: channels 16 tile + 4 q + r
      const int j = 16 * tile + 4 * q + r;
      b2[r] = j < C ? b2p[j] : 0.0f;
      w3[r] = j < C ? w3p[j] : 0.0f;
    }
  }
  const float b3 = wf[P - 1];
  // this thread's share of the first layer: channels 4 cg .. + 4 of every
  // (T / groups)-th position (consecutive lanes store consecutive positions)
  const int groups = C / 4, per = T / groups;
  const int cg = tid / per, p0 = tid - cg * per;
  const bool first = cg < groups;  // not the threads past the last whole group
  for (int c = tid; c < C; c += T)
    w1s[c] = make_float4(wf[3 * c], wf[3 * c + 1], wf[3 * c + 2], wf[3 * C + c]);
  // query i of this work-group's share: its row, and its list entry
  auto entry = [&](int64_t i) { return a.plist ? a.plist[f * a.stride + i] : i; };
  // Query j of the share: its row in xs slot j mod 3, its planes in slot j mod
  // 2, its flag in slot j mod 4 (a flag is read in iteration j, cleared in the
  // next, and set again two barriers later at the earliest).
  auto stage_row = [&](int64_t e, int j) {
    const float *xr = a.x + (a.plist ? e / a.N : e) * m;
    for (int p = tid; p < m; p += T) xs[(j % 3) * xrow + p + 1] = xr[p];
  };
  auto first_layer = [&](int j) {
    const float *xp = xs + (j % 3) * xrow;
    uint16_t *pl = planes + 3 * (j & 1) * plane;
    SplitRange range;
    if (first)
      for (int p = p0; p < m; p += per) {
        const float4 v = make_float4(conv_first(w1s[4 * cg], xp, p), conv_first(w1s[4 * cg + 1], xp, p),
                                     conv_first(w1s[4 * cg + 2], xp, p), conv_first(w1s[4 * cg + 3], xp, p));
        split_store4(v, pl, plane, (cg >> 1) * rows8 + 8 * (p + 1) + 4 * (cg & 1), range);
      }
    if (range.exceeded()) bad[j & 3] = 1;
  };
  auto write_out = [&](int64_t e, int j) {
    float y = 0.0f;
    for (int w = 0; w < T / kWave; ++w) y += red[(j & 1) * (T / kWave) + w];
    y = y / static_cast<float>(m) + b3;
    if (a.plist) a.dfo[e] = y - a.offsets[static_cast<int64_t>(a.pair[e / a.N]) * a.F + f];
    else a.out[e * a.F + f] = y;
  };
  const int64_t step = gridDim.y;
  int64_t i = blockIdx.y, e_cur = entry(i), e_prev = -1;
  __syncthreads();
  if (oddw) bad[4] = 1;
  stage_row(e_cur, 0);
  __syncthreads();
  first_layer(0);
  int j = 0;
  for (; i < n; i += step, ++j) {
    const int64_t e_next = i + step < n ? entry(i + step) : -1;
    if (e_next >= 0) stage_row(e_next, j + 1);
    __syncthreads();  // query j's planes, the next row and query j - 1's sums are complete
    if (e_prev >= 0 && tid == 0) write_out(e_prev, j - 1);
    const bool plain = (bad[j & 3] | bad[4]) != 0;  // uniform
    if (tid == 0 && j > 0) bad[(j - 1) & 3] = 0;
    if (e_next >= 0) first_layer(j + 1);
    float part = 0.0f;
    if (plain) {
      part = conv_plain(wf, m, C, w1s, xs + (j % 3) * xrow);
    } else {
      const uint16_t *pl = planes + 3 * (j & 1) * plane;
      float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      for (int nt = pg; 16 * nt < m; nt += a.ng) {
        floatx4 hi = {0.0f, 0.0f, 0.0f, 0.0f}, lo = hi;
        const uint16_t *bp = pl + q * rows8 + 8 * (16 * nt + col);  // position p - 1 is stored at p
#pragma unroll
        for (int k = 0; k < KS; ++k) {
          const uint16_t *at = bp + 8 * (k % 3) + 4 * (k / 3) * rows8;
          const bf16x8 x0 = *reinterpret_cast<const bf16x8 *>(at);
          const bf16x8 x1 = *reinterpret_cast<const bf16x8 *>(at + plane);
          const bf16x8 x2 = *reinterpret_cast<const bf16x8 *>(at + 2 * plane);
          lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[k][2], x0, lo, 0, 0, 0);
          hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[k][0], x0, hi, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[k][1], x0, lo, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[k][1], x1, lo, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[k][0], x1, lo, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[k][0], x2, lo, 0, 0, 0);
        }
        const bool in = 16 * nt + col < m;
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] += in ? fmaxf(hi[r] + lo[r] + b2[r], 0.0f) : 0.0f;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) part = fmaf(w3[r], sum[r], part);
    }
    part = wave_sum(part);
    if (lane == 0) red[(j & 1) * (T / kWave) + wave] = part;
    e_prev = e_cur;
    e_cur = e_next;
  }
  __syncthreads();
  if (tid == 0) write_out(e_prev, j - 1);
}

template <int KS>
void conv_launch(const ConvArgs &a, dim3 grid, int waves, hipStream_t st) {
  const size_t lds = conv_lds(a.m, a.C, KS, waves, a.bufs);
  auto kern = k_cnn_infer_split<KS>;
  allow_lds(reinterpret_cast<const void *>(kern), lds);
  hipLaunchKernelGGL(kern, grid, dim3(kWave * waves), lds, st, a);
  LAUNCH_OK("cnn_infer_split");
}

}  // namespace

// Up to 128 channels and 256 positions whose planes fit in LDS; false, with
// nothing launched, otherwise.  Wavefronts: one per 16 output channels, times
// as many position groups as 12 wavefronts (8 above 96 channels, whose parts
// take twice the registers) and the positions allow.  With more filters than CUs
// and up to 64 channels the 12 are dealt to as many work-groups as there are
// filters per CU and their planes fit its LDS: a work-group with a CU to itself
// leaves it idle while it waits for the weights and at the barriers.  One query
// and 100, plain kernel, 12 wavefronts, this: 300 filters of 64 channels x 64
// positions 27, 45, 19 us and 1,326, 431, 289; 1,024 of 20 x 40 9.7, 19.6, 10.1 and
// 475, 506, 232; 8,192 of 32 x 96 121, 387, 96 and (20 queries) 1,495, 1,336, 680.
// Not for 96 channels (300 x 48 positions, 100 queries: 626 and 642).  All of
// it follows from the filters alone: the position groups are the order of a sum.
//
// Work-groups share a filter's queries like the MLP inference's, the read of the
// weights standing for two queries; those with one query each have one set of
// planes, which lets more of them share a CU.
bool launch_cnn_infer_split(const float *w, int F, int m, int C, const float *x, int64_t nq, float *out,
                            const int64_t *plist, const int32_t *pcnt, int64_t stride, int N, const int32_t *pair,
                            const float *offsets, float *dfo, hipStream_t st) {
  const int ks = 3 * ((C + 31) / 32);
  if (C > 128 || m > 256) return false;
  ConvArgs a{w, F, m, C, x, nq, out, plist, pcnt, stride, N, pair, offsets, dfo, 0, 0, 2};
  a.mt = (C + 15) / 16;
  int most = ks <= 9 ? kConvMaxWaves : 8;
  if (ks <= 6) {
    const int64_t fit = 160 * 1024 / conv_lds(m, C, ks, most, 2);
    const int64_t per_cu = std::min({ceil_div(F, device_cus()), fit, static_cast<int64_t>(most / a.mt)});
    most /= static_cast<int>(std::max<int64_t>(1, per_cu));
  }
  a.ng = std::max(1, std::min(most / a.mt, (m + 15) / 16));
  const int waves = a.mt * a.ng;
  if (conv_lds(m, C, ks, waves, 2) > 160 * 1024) return false;
  const int64_t n = plist ? ceil_div(stride, 8) : nq;
  int share = 1;
  int64_t best = 0;
  for (int c = 1; c <= 16 && c <= n; ++c) {
    const int64_t cost = ceil_div(static_cast<int64_t>(F) * c, device_cus()) * (2 + ceil_div(n, c));
    if (best == 0 || cost < best) {
      best = cost;
      share = c;
    }
  }
  if (!plist && nq <= share) a.bufs = 1;
  const dim3 grid(F, share);
  switch (ks) {
    case 3: conv_launch<3>(a, grid, waves, st); break;
    case 6: conv_launch<6>(a, grid, waves, st); break;
    case 9: conv_launch<9>(a, grid, waves, st); break;
    default: conv_launch<12>(a, grid, waves, st); break;
  }
  return true;
}

}  // namespace leafi
