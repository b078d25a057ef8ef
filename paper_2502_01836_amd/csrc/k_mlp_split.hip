// MLP filter inference on the bf16 matrix cores at FP32 accuracy, for up to
// 256 inputs and 256 hidden units (any multiples of 4).
//
// Every FP32 operand is split into three bf16 parts, v = v0 + v1 + v2 (each
// part the rounded remainder of the ones before, 24 bits in all), and a
// product keeps the six terms of its parts down to 2^-18 of it: x0 w0, x0 w1,
// x1 w0, x1 w1, x0 w2, x2 w0; the terms left out are 2^-26 of it.  The parts'
// products are exact and are accumulated in FP32, the leading term apart from
// the corrections, so the result's error stays that of FP32 accumulation
// (measured against 64 bits on 1,024 filters 256 -> 256 -> 1: 7.7e-8 relative,
// FP32 matrix products 7.8e-8).  Six v_mfma_f32_16x16x32_bf16 replace eight
// v_mfma_f32_16x16x4_f32, which take 2.7 times as long.
//
// A work-group of eight wavefronts, or four, takes one filter and every gridDim.y-th
// batch of its rows (all queries, or the filter's listed (query, leaf)
// pairs).  The filter's W1 is read once and kept as bf16 parts in registers:
// wavefront w holds the HT 16-unit hidden tiles of hidden group w mod wh for
// all inputs and computes the 16-row tiles of row group w / wh.  A batch's
// rows are read one batch ahead, straight into LDS, split once by the whole
// work-group into three LDS planes (row stride 8 elements past the inputs, so
// the 16 rows of an operand read start in different banks), and read from
// there as the B operand.  With m = h = 256 the parts of W1 take 192 of a
// lane's 256 registers: one work-group per CU, two wavefronts per SIMD.  With
// more filters than CUs, narrow ones are dealt to work-groups of half the size,
// two and more per CU, whose waits overlap: the read and split of a filter's W1
// is most of a small call.
// What bounds it is the matrix cores (45 % of the wavefronts' cycles, at the
// clock the chip holds under them), then the split and the two barriers of a
// batch, and the read of W1 at its start.  1,024 filters x 500 rows, m = h =
// 256: 720 -> 402 us (167 TFLOP/s of FP32 products; the FP32 matrix rate is
// 151); the 6.6M pairs of a 2,198-filter 96 -> 96 -> 1 batch: 3.9 -> 1.2 ms,
// where the FP32 kernel had three of its eight wavefronts at work.
//
// A row that holds an infinity, a NaN or an operand out of the parts' range
// (split_bf16.h) is evaluated with plain FP32 arithmetic instead, and with such
// a weight every row of its filter.  The
// other rows of its batch keep the matrix products' values (an operand column
// reaches its own output column alone): what a row's prediction is does not
// depend on the rows beside it.
#include <algorithm>

#include "device_util.h"
#include "kernels.h"
#include "split_bf16.h"

namespace leafi {

namespace {

constexpr int kSplitWaves = 8;  // most wavefronts of a work-group (4 or 8)
constexpr int kSplitPre = 6;    // 16-byte pieces of a batch per thread: of eight wavefronts, rows x padded inputs <= 12,288

struct SplitArgs {
  const float *w;
  int F, m, h;
  const float *x;
  int64_t nq;       // dense form (plist null): rows, out[r F + f] = d^f
  float *out;
  const int64_t *plist;  // listed form: entries e = q N + visit position
  const int32_t *pcnt;
  int64_t stride;
  int N;
  const int32_t *pair;
  const float *offsets;
  float *dfo;       // dfo[e] = d^f - offsets[pair[q] F + f]
  int wh, wr, rt;   // hidden groups, row groups, 16-row tiles per row group and batch
};

// Requests 16 bytes per active lane from p straight into LDS: lane l's land at
// base + 16 l (base uniform, within the first 64 KiB of LDS).  Written in
// assembly because the compiler, which cannot tell the parts of a dynamic LDS
// block apart, would otherwise wait for these loads before any LDS read.
__device__ __forceinline__ void load_to_lds(const float *p, const float *base) {
  const uint32_t at = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) float *)base));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(
                   __builtin_amdgcn_readfirstlane(at)),
               "v"(p)
               : "memory", "m0");
}
// Until every load this wavefront requested, into LDS or registers, has landed.
__device__ __forceinline__ void wait_lds_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Plain FP32 evaluation of the batch's flagged rows, or with `all` of every
// row, one wavefront per row: row sums into red (the other hidden groups' sums
// zero), the flags back to 0.
__device__ __forceinline__ void split_plain_rows(const float *__restrict__ wf, int m, int h, const float *__restrict__ x,
                                              const int64_t *rowq, int *rowbad, bool all, int nr, int rb, int wh,
                                              float *red) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const float *b1 = wf + static_cast<int64_t>(h) * m, *w2 = b1 + h;
  for (int c = wave; c < nr; c += blockDim.x / kWave) {
    if (!all && rowbad[c] == 0) continue;  // uniform
    const float *xr = x + rowq[c] * m;
    float p = 0.0f;
    for (int j = lane; j < h; j += kWave) {
      float z = 0.0f;
      for (int i = 0; i < m; ++i) z = fmaf(xr[i], wf[static_cast<int64_t>(i) * h + j], z);
      p = fmaf(w2[j], fmaxf(z + b1[j], 0.0f), p);
    }
    p = wave_sum(p);
    if (lane == 0) {
      rowbad[c] = 0;
      for (int g = 0; g < wh; ++g) red[g * rb + c] = g == 0 ? p : 0.0f;
    }
  }
}

// LDS of a work-group: the next batch's rows, the planes, b1 and w2 (padded hidden units), the
// hidden groups' row sums (two batches), the batch's query rows and list
// entries (two batches), its row flags, four flags.
__host__ __device__ inline int split_rows(const SplitArgs &a) { return 16 * a.wr * a.rt; }
size_t split_lds(const SplitArgs &a, int ks, int ht) {
  const size_t rb = split_rows(a);
  return rb * a.m * 4 + 3 * rb * (32 * ks + 8) * 2 + 2 * static_cast<size_t>(16 * ht * a.wh) * 4 + 2 * a.wh * rb * 4 + 4 * rb * 8 + rb * 4 + 16;
}

template <int KS, int HT, int NW>
__global__ void __launch_bounds__(kWave * NW, 2) k_mlp_infer_split(SplitArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int kSplitThreads = kWave * NW;
  constexpr int MP = 32 * KS + 8;  // row stride of the planes
  const int f = blockIdx.x;
  const int64_t n = a.plist ? static_cast<int64_t>(a.pcnt[f]) : a.nq;
  const int rb = split_rows(a);
  const int64_t nb = (n + rb - 1) / rb;
  if (static_cast<int64_t>(blockIdx.y) >= nb) return;  // uniform
  const int m = a.m, h = a.h, m4 = m / 4, wh = a.wh, wr = a.wr;
  const int plane = rb * MP, hp = 16 * HT * wh;
  float *raw = reinterpret_cast<float *>(smem);           // [rb][m], the next batch's rows
  uint16_t *planes = reinterpret_cast<uint16_t *>(raw + rb * m);  // [3][rb][MP]
  float *b1s = reinterpret_cast<float *>(planes + 3 * plane);  // [hp]
  float *w2s = b1s + hp;                                       // [hp]
  float *red = w2s + hp;                                       // [2][wh][rb]
  int64_t *rowq = reinterpret_cast<int64_t *>(red + 2 * wh * rb);  // [2][rb]
  int64_t *rent = rowq + 2 * rb;                                   // [2][rb]
  int *rowbad = reinterpret_cast<int *>(rent + 2 * rb);            // [rb] the batch's rows for plain arithmetic
  int *bad = rowbad + rb;                                          // [2] batch holds such rows, [1] weights
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 15, q = lane >> 4;
  const int hg = wave % wh, rg = wave / wh;
  const int64_t P = static_cast<int64_t>(h) * m + 2 * h + 1;
  const float *wf = a.w + f * P;
  // the rows of batch b into slot s (threads below rb)
  auto find_rows = [&](int64_t b, int s) {
    if (tid < rb) {
      const int64_t i = b * rb + tid;
      int64_t qr = -1, e = -1;
      if (b < nb && i < n) {
        if (a.plist) {
          e = a.plist[f * a.stride + i];
          qr = e / a.N;
        } else {
          qr = i;
        }
      }
      rowq[s * rb + tid] = qr;
      rent[s * rb + tid] = e;
    }
  };
  int64_t b = blockIdx.y;
  find_rows(b, 0);
  for (int e = tid; e < rb + 4; e += kSplitThreads) rowbad[e] = 0;  // and bad
  // inputs past m are zero in every row and in W1
  if (m < 32 * KS)
    for (int e = tid; e < 3 * rb * (32 * KS - m); e += kSplitThreads) {
      const int r = e / (32 * KS - m);
      planes[r * MP + m + e - r * (32 * KS - m)] = 0;
    }
  for (int j = tid; j < hp; j += kSplitThreads) {
    b1s[j] = j < h ? wf[static_cast<int64_t>(h) * m + j] : 0.0f;
    w2s[j] = j < h ? wf[static_cast<int64_t>(h) * m + h + j] : 0.0f;
  }
  const float b2 = wf[P - 1];
  __syncthreads();
  // Piece u of this thread in a batch: row e4 / m4, 4-input group e4 mod m4
  // (e4 < 3,072, so the reciprocal's error stays below 1 / m4).  Derived from
  // an opaque thread number each time: kept across the loop, the pieces'
  // addresses would push parts of W1 out of the registers.
  const uint32_t inv4 = ((1u << 20) + m4 - 1) / m4;
  auto my_thread = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  auto fetch = [&](int s) {
    const int t = my_thread();
#pragma unroll
    for (int u = 0; u < kSplitPre; ++u) {
      const int e4 = t + u * kSplitThreads;
      const int c = static_cast<int>((static_cast<uint32_t>(e4) * inv4) >> 20);
      if (c < rb) {
        const int64_t r = rowq[s * rb + c];
        if (r >= 0) load_to_lds(a.x + r * m + 4 * (e4 - c * m4), raw + 4 * (64 * wave + u * kSplitThreads));
      }
    }
  };
  // W1's parts: lane holds hidden unit 16 (HT hg + t) + col, inputs 32 ks + 8 q .. + 8
  bf16x8 W[HT][KS][3];
  {
    // every load in flight before the first is split: the raw values of the
    // steps to come and the parts of those done never outnumber the parts
    float raw[KS][HT][8];
    if (m == 32 * KS && h == hp) {  // uniform: no padding
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < HT; ++t) {
          const uint32_t at = static_cast<uint32_t>(32 * ks + 8 * q) * h + 16 * (HT * hg + t) + col;
#pragma unroll
          for (int e = 0; e < 8; ++e) raw[ks][t][e] = wf[at + static_cast<uint32_t>(e) * h];
        }
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < HT; ++t) {
          const int j = 16 * (HT * hg + t) + col;
          const uint32_t at = static_cast<uint32_t>(32 * ks + 8 * q) * h + j;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const bool in = j < h && 32 * ks + 8 * q + e < m;
            const float y = wf[in ? at + static_cast<uint32_t>(e) * h : 0u];
            raw[ks][t][e] = in ? y : 0.0f;
          }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    bool odd = false;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < HT; ++t) odd |= split8(raw[ks][t], W[t][ks][0], W[t][ks][1], W[t][ks][2]);
    if (rg < wr && odd) bad[2] = 1;
  }
  fetch(0);
  int nr_prev = 0;
  auto write_out = [&](int s, int nr) {
    if (tid < nr) {
      float y = b2;
      for (int g = 0; g < wh; ++g) y += red[(s * wh + g) * rb + tid];
      const int64_t r = rowq[s * rb + tid];
      if (a.plist) a.dfo[rent[s * rb + tid]] = y - a.offsets[static_cast<int64_t>(a.pair[r]) * a.F + f];
      else a.out[r * a.F + f] = y;
    }
  };
  int s = 0;
  for (; b < nb; b += gridDim.y, s ^= 1) {
    const int nr = static_cast<int>(n - b * rb < rb ? n - b * rb : rb);
    __syncthreads();  // the planes and the other slot's sums are complete
    write_out(s ^ 1, nr_prev);
    wait_lds_loads();  // each thread splits the pieces its own wavefront requested
    SplitRange range;
    {
      const int t = my_thread();
#pragma unroll
      for (int u = 0; u < kSplitPre; ++u) {
        const int e4 = t + u * kSplitThreads;
        const int c = static_cast<int>((static_cast<uint32_t>(e4) * inv4) >> 20);
        if (c < nr) {
          const float4 v = *reinterpret_cast<const float4 *>(raw + 4 * e4);
          split_store4(v, planes, plane, c * MP + 4 * (e4 - c * m4), range);
        }
      }
    }
    if (range.exceeded()) {  // rare: which of the thread's pieces
      bad[s] = 1;
      for (int e4 = tid; e4 / m4 < nr; e4 += kSplitThreads) {
        SplitRange piece;
        split_store4(*reinterpret_cast<const float4 *>(raw + 4 * e4), planes, plane, e4 / m4 * MP + 4 * (e4 % m4), piece);
        if (piece.exceeded()) rowbad[e4 / m4] = 1;
      }
    }
    find_rows(b + gridDim.y, s ^ 1);
    __syncthreads();
    fetch(s ^ 1);
    const bool all = bad[2] != 0, some = bad[s] != 0;  // uniform
    if (rg < wr && !all) {
      for (int rt = 0; rt < a.rt; ++rt) {
        const int row0 = 16 * (rg + wr * rt);
        if (row0 >= nr) break;  // uniform
        floatx4 hi[HT], lo[HT];
#pragma unroll
        for (int t = 0; t < HT; ++t) hi[t] = lo[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        const uint16_t *xp = planes + (row0 + col) * MP + 8 * q;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8 x0 = *reinterpret_cast<const bf16x8 *>(xp + 32 * ks);
          const bf16x8 x1 = *reinterpret_cast<const bf16x8 *>(xp + plane + 32 * ks);
          const bf16x8 x2 = *reinterpret_cast<const bf16x8 *>(xp + 2 * plane + 32 * ks);
          // the hidden tiles take turns, so consecutive products do not wait on each other
#define LEAFI_TERM(acc, wp, xv)                                                                       \
  _Pragma("unroll") for (int t = 0; t < HT; ++t) acc[t] =                                             \
      __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[t][ks][wp], xv, acc[t], 0, 0, 0);
          LEAFI_TERM(lo, 2, x0)
          LEAFI_TERM(hi, 0, x0)
          LEAFI_TERM(lo, 1, x0)
          LEAFI_TERM(lo, 1, x1)
          LEAFI_TERM(lo, 0, x1)
          LEAFI_TERM(lo, 0, x2)
#undef LEAFI_TERM
        }
        // lane holds hidden units 4 q + r of each tile for row `col`
        float p = 0.0f;
#pragma unroll
        for (int t = 0; t < HT; ++t) {
          const int j = 16 * (HT * hg + t) + 4 * q;
          const float4 b1 = *reinterpret_cast<const float4 *>(b1s + j);
          const float4 w2 = *reinterpret_cast<const float4 *>(w2s + j);
          p = fmaf(w2.x, fmaxf(hi[t][0] + lo[t][0] + b1.x, 0.0f), p);
          p = fmaf(w2.y, fmaxf(hi[t][1] + lo[t][1] + b1.y, 0.0f), p);
          p = fmaf(w2.z, fmaxf(hi[t][2] + lo[t][2] + b1.z, 0.0f), p);
          p = fmaf(w2.w, fmaxf(hi[t][3] + lo[t][3] + b1.w, 0.0f), p);
        }
        p += __shfl_xor(p, 16, kWave);
        p += __shfl_xor(p, 32, kWave);
        if (lane < 16) red[(s * wh + hg) * rb + row0 + lane] = p;
      }
    }
    if (all || some) {
      __syncthreads();  // the flagged rows' own sums replace the products'
      split_plain_rows(wf, m, h, a.x, rowq + s * rb, rowbad, all, nr, rb, wh, red + s * wh * rb);
    }
    if (tid == 0) bad[s ^ 1] = 0;  // the next batch's (set only after the next barrier)
    nr_prev = nr;
  }
  __syncthreads();
  write_out(s ^ 1, nr_prev);
}

template <int KS, int HT>
void split_launch(const SplitArgs &a, int waves, dim3 grid, hipStream_t st) {
  const size_t lds = split_lds(a, KS, HT);
  auto kern = waves == 4 ? k_mlp_infer_split<KS, HT, 4> : k_mlp_infer_split<KS, HT, kSplitWaves>;
  allow_lds(reinterpret_cast<const void *>(kern), lds);
  hipLaunchKernelGGL(kern, grid, dim3(kWave * waves), lds, st, a);
  LAUNCH_OK("mlp_infer_split");
}

template <int KS>
void split_launch_ht(int ht, const SplitArgs &a, int waves, dim3 grid, hipStream_t st) {
  if constexpr (KS <= 3)
    if (ht == 4) return split_launch<KS, 4>(a, waves, grid, st);
  if constexpr (KS <= 4)
    if (ht == 3) return split_launch<KS, 3>(a, waves, grid, st);
  if (ht == 2) return split_launch<KS, 2>(a, waves, grid, st);
  split_launch<KS, 1>(a, waves, grid, st);
}

}  // namespace

// The arrangement of eight wavefronts: HT hidden tiles per wavefront (as many
// as its 256 registers hold the parts and accumulators of) in wh hidden groups
// x wr row groups, by the row tiles finished per unit of time (wr / HT), then by
// more hidden tiles (each operand read from LDS serves more products).  With
// listed pairs, whose numbers only the device knows, an eighth of the queries
// stands for a filter's rows.
//
// Four wavefronts hold the same HT and wh, so the same sums, with fewer row
// groups, where there are more filters than CUs and up to four hidden groups,
// as many rows at a time as let a second work-group share the CU's LDS: for up
// to 128 inputs (1,024 filters 96 -> 96: one row 33 -> 17 us, 500 rows 96 -> 84;
// the FP32 kernel that kept W1 in registers 20 and 271), above that, where the
// batches would be of 16 rows, for dense calls of up to 32 (256 -> 64, one row: 34 ->
// 18 us).
//
// Which filters are evaluated here follows from the filters alone (their
// number and sizes), never from the rows of a call: a prediction's bits are
// the same in any batch, and the same in a calibration (dense) as in the
// search that tests its offset (listed).  Few filters are left to the FP32
// kernels' tiles of 32 rows, which need not read and split all of W1 (about 15
// us) first (3 filters 240 -> 152, 35 rows: 12.6 us, here 18.5; 128 of 256 ->
// 256: 14 and 20 for 40 rows, 90 and 57 for 500), and so are wide ones whose
// sizes pad its 16 x 16 tiles (300 of 228 -> 144: 31 and 39 for 40 rows, 175 and
// 151 for 500).  From a filter per CU on the rest is the faster here: 256
// -> 256, 256 filters, one row 25 us (the FP32 kernel that kept W1 in registers)
// and 19, 500 rows 178 and 99.
bool launch_mlp_infer_split(const float *w, int F, int m, int h, const float *x, int64_t nq, float *out,
                            const int64_t *plist, const int32_t *pcnt, int64_t stride, int N, const int32_t *pair,
                            const float *offsets, float *dfo, bool small_batches, hipStream_t st) {
  if (F < device_cus() || m > 256 || h > 256 || m % 4 != 0 || reinterpret_cast<uintptr_t>(x) % 16 != 0) return false;
  const int ks = (m + 31) / 32, ht_all = (h + 15) / 16, tiles = 24 / ks;
  SplitArgs a{w, F, m, h, x, nq, out, plist, pcnt, stride, N, pair, offsets, dfo, 0, 0, 0};
  int ht = 0;
  for (int c = ks <= 3 ? 4 : ks == 4 ? 3 : 2; c >= 1; --c) {
    const int wh = (ht_all + c - 1) / c;
    if (wh > kSplitWaves) continue;
    const int wr = std::min(kSplitWaves / wh, tiles);
    if (ht == 0 || wr * ht > a.wr * c) {
      ht = c;
      a.wh = wh;
      a.wr = wr;
    }
  }
  const bool narrow = ks <= 4 && a.wh <= 4;
  if (!narrow && (m % 16 != 0 || h % 16 != 0)) return false;
  a.rt = small_batches ? 1 : std::max(1, std::min(3, tiles / a.wr));
  int waves = kSplitWaves;
  if (F > device_cus() && a.wh <= 4 && (ks <= 4 || (!plist && nq <= 32))) {
    waves = 4;
    a.wr = std::min(waves / a.wh, tiles);
    a.rt = small_batches ? 1 : std::min(3, tiles / a.wr);
  }
  if (!plist) {  // no LDS for rows that a call does not have
    const int need = static_cast<int>(std::min<int64_t>(ceil_div(nq, 16), tiles));
    a.wr = std::min(a.wr, need);
    a.rt = std::min<int>(a.rt, ceil_div(need, a.wr));
  }
  auto fits = [&] {
    return split_rows(a) * m / 4 <= kSplitPre * kWave * waves && (waves == kSplitWaves || split_lds(a, ks, ht) <= 80 * 1024);
  };
  while (!fits()) --(a.rt > 1 ? a.rt : a.wr);
  // how many work-groups share a filter: rounds of the chip x (the read of W1,
  // about three batches' time, and the batches of one)
  const int64_t nb = std::max<int64_t>(1, ceil_div(plist ? ceil_div(stride, 8) : nq, split_rows(a)));
  int share = 1;
  int64_t best = 0;
  for (int c = 1; c <= 16 && c <= nb; ++c) {
    const int64_t cost = ceil_div(static_cast<int64_t>(F) * c, device_cus()) * (3 + ceil_div(nb, c));
    if (best == 0 || cost < best) {
      best = cost;
      share = c;
    }
  }
  const dim3 grid(F, share);
  switch (ks) {
    case 1: split_launch_ht<1>(ht, a, waves, grid, st); break;
    case 2: split_launch_ht<2>(ht, a, waves, grid, st); break;
    case 3: split_launch_ht<3>(ht, a, waves, grid, st); break;
    case 4: split_launch_ht<4>(ht, a, waves, grid, st); break;
    case 5: split_launch_ht<5>(ht, a, waves, grid, st); break;
    case 6: split_launch_ht<6>(ht, a, waves, grid, st); break;
    case 7: split_launch_ht<7>(ht, a, waves, grid, st); break;
    default: split_launch_ht<8>(ht, a, waves, grid, st); break;
  }
  return true;
}

}  // namespace leafi
