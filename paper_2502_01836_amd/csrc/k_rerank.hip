// Per-item rerank of a round's candidate lists and the per-query bound that
// lets a search round skip items and candidates (SearchNode of Algorithm 2:
// the result update after a leaf's scan).
//
// After a pass's scan every (query, tile) list holds its kprime best keys
// (truncated BF16 or FP32 squared distances with rows).  k_query_bound finds
// per query an upper bound U of its k-th distance after the round, then
// certifies the query's items whose every candidate is provably beyond U and
// lists the rest; k_item_rerank merges each listed item's chunk lists
// and reranks its candidates in FP32 (FP64 within the error band of the k-th),
// writing the item's exact top-k and the bound that certifies the rest.
#include <algorithm>

#include "device_util.h"
#include "kernels.h"
#include "scan_bounds.h"
#include "wave_sort.h"

namespace leafi {

namespace {

// Selection instead of a full sort when at most kSelectMax of at most
// 64 * kSelectPerLane chunk candidates are wanted.
constexpr int kSelectMax = 16;
constexpr int kSelectPerLane = 16;

// One wavefront per item.  LDS: merged keys [P], then per candidate the fp32
// key, FP64 distance and row.
// The kp smallest of an item's n chunk-list keys (kprime slots per chunk)
// into buf (ascending, kKeyMax past the last real key): kp rounds of a
// the keys above the previous one (keys are unique), U per lane in registers
// (unconditional loads of clamped entries, so all of a lane's loads are in
// flight together; n >= kprime >= kp >= 1, so entry 0 exists; n <= 64 U).
template <int U>
__device__ inline void select_keys(const uint64_t *__restrict__ cand, int64_t t0, int G, int g, int mq, int j,
                                   int kprime, int kp, int n, int lane, uint64_t *buf) {
  uint64_t mine[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = lane + u * kWave;
    const int ec = e < n ? e : 0;
    const int c = ec / kprime;
    const uint64_t v = cand[((t0 + static_cast<int64_t>(c) * G + g) * mq + j) * kprime + (ec - c * kprime)];
    mine[u] = e < n ? v : kKeyMax;
  }
  uint64_t prev = 0;
  bool first = true;
  for (int r = 0; r < kp; ++r) {
    uint64_t lo = kKeyMax;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if ((first || mine[u] > prev) && mine[u] < lo) lo = mine[u];
    lo = wave_min_u64(lo);
    if (lane == 0) buf[r] = lo;
    prev = lo;
    first = false;
    if (lo == kKeyMax) {  // no keys left: the rest stay empty
      for (int e = r + 1 + lane; e < kp; e += kWave) buf[e] = kKeyMax;
      break;
    }
  }
}

// ---- a query's bound for the rerank --------------------------------------------
//
// After a search round's BF16 scan, every candidate list of a query is sorted
// by key (bf16 squared distance, row).  The k smallest keys over all of them
// belong to k distinct rows, each no farther than sqrt(key + delta16) + eps_q
// + eps_L, so the query's k-th exact distance after this round's merge is at
// most U = sqrt(kth key + delta16) + eps_q + max_L eps_L (and at most its tau
// before the round).  A candidate whose lower bound sqrt(key - delta16) -
// eps_q - eps_L exceeds U can never enter the query's top k, so the rerank
// skips its FP32 and FP64 distances.  The k-th smallest key is found by a
// tournament over the list heads, 64 x kBoundSlots lists per pass; a pass
// keeps the k smallest so far in LDS for the next, and each round emits the
// run of those below the lists' smallest head (up to 64 at once) or that
// head.
constexpr int kBoundSlots = 4;

__device__ inline int bound_pass(int64_t q, int N, int k, int kprime, int mq, int chunk, int cmax, const RoundBufs &b,
                                 const StoreView &s, const uint64_t *__restrict__ cand, int l0, int nl,
                                 const uint64_t *in, int n_in, uint64_t *out, int lane) {
  uint64_t hd[kBoundSlots], n1[kBoundSlots], n2[kBoundSlots];
  int64_t base[kBoundSlots];
  int pos[kBoundSlots], cnt[kBoundSlots];
  const int kp = item_kprime(b.kp_query, kprime, k, true);
#pragma unroll
  for (int i = 0; i < kBoundSlots; ++i) {
    const int lam = l0 + lane + kWave * i;
    cnt[i] = 0;
    base[i] = 0;
    if (lam < l0 + nl) {
      const int r = lam / cmax, c = lam - r * cmax;
      const int idx = b.qitem_idx[q * N + r];
      const int L = b.item_leaf[idx];
      const int ist0 = b.leaf_istart[L], ist1 = b.leaf_istart[L + 1];
      const int C = static_cast<int>((s.leaf_off[L + 1] - s.leaf_off[L] + chunk - 1) / chunk);
      if (c < C) {
        const int p = idx - ist0, g = p / mq, j = p - g * mq, G = (ist1 - ist0 + mq - 1) / mq;
        base[i] = (tile_of(b.tile_start, L, g, c, G) * mq + j) * kprime;
        cnt[i] = kp;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kBoundSlots; ++i) {
    hd[i] = cnt[i] > 0 ? cand[base[i]] : kKeyMax;
    n1[i] = cnt[i] > 1 ? cand[base[i] + 1] : kKeyMax;
    n2[i] = cnt[i] > 2 ? cand[base[i] + 2] : kKeyMax;
    pos[i] = 3;
  }
  int o = 0, rp = 0;
  while (o < k) {
    uint64_t lo = kKeyMax;
#pragma unroll
    for (int i = 0; i < kBoundSlots; ++i) lo = hd[i] < lo ? hd[i] : lo;
    const uint64_t g = wave_min_u64(lo);
    // the running list's keys below the lists' smallest head come next, as
    // one run (lane j checks entry rp + j)
    const bool below = rp + lane < n_in && o + lane < k && in[rp + lane] < g;
    const uint64_t bm = __ballot(below);
    const int run = ~bm == 0 ? kWave : __builtin_ctzll(~bm);
    if (run > 0) {
      if (lane < run) out[o + lane] = in[rp + lane];
      o += run;
      rp += run;
      continue;
    }
    if (g == kKeyMax) break;  // every list is exhausted
    if (lane == 0) out[o] = g;
    ++o;
    if (rp < n_in && in[rp] == g) ++rp;
#pragma unroll
    for (int i = 0; i < kBoundSlots; ++i) {
      if (hd[i] == g) {  // the row may sit in two lists (a leaf rescanned): every copy advances
        hd[i] = n1[i];
        n1[i] = n2[i];
        n2[i] = pos[i] < cnt[i] ? cand[base[i] + pos[i]] : kKeyMax;
        ++pos[i];
      }
    }
  }
  wave_lds_sync();
  return o;
}

// One item of a search round: each chunk list is sorted, so its first key is
// its smallest, and every row of the item has a key at least the smallest of
// them (or was never a candidate: key >= the tau threshold).  When even that
// bound exceeds the query's bound U, no row of the item can enter the query's
// top k: the item contributes nothing and is certified by that bound (no
// sort, no rerank).  Returns whether the item still needs its rerank.
__device__ inline bool item_live_after_bound(const StoreView &s, const QueryView &qv, const RoundBufs &b, int mq,
                                             int kprime, const uint64_t *__restrict__ cand, int item, int64_t q,
                                             float U) {
  const int m = s.m;
  const int L = b.item_leaf[item];
  const int ist0 = b.leaf_istart[L], ist1 = b.leaf_istart[L + 1];
  const int64_t off0 = s.leaf_off[L], off1 = s.leaf_off[L + 1];
  const float tau_q = b.tau[q], qn_q = qv.qn16[q], qe_q = qv.qeps[q], le_L = s.leaf_eps[L];
  const int64_t t0 = b.tile_start[L];
  const int pos = item - ist0;
  const int g = pos / mq, j = pos - g * mq;
  const int C = static_cast<int>((off1 - off0 + b.chunk - 1) / b.chunk);
  const int G = (ist1 - ist0 + mq - 1) / mq;
  uint64_t h = kKeyMax;
  for (int c = 0; c < C; ++c) {
    const uint64_t v = cand[((t0 + static_cast<int64_t>(c) * G + g) * mq + j) * kprime];
    h = v < h ? v : h;
  }
  float kd = h != kKeyMax ? key_d2(h) : __builtin_inff();
  kd = fminf(kd, tau_threshold(tau_q, qn_q, qe_q, le_L, m));
  double lower = -1.0;
  if (kd < __builtin_inff()) {
    const double v = static_cast<double>(kd) - bf16_delta(qn_q, m);
    lower = (v > 0.0 ? sqrt(v) : 0.0) - qe_q - le_L;
  }
  if (lower > static_cast<double>(U)) {
    float lb = static_cast<float>(lower);
    if (static_cast<double>(lb) > lower) lb = nextafterf(lb, -__builtin_inff());
    b.item_cnt[item] = 0;
    b.item_bound[item] = lb;
    return false;
  }
  return true;
}

// One work-group per query: its four wavefronts take every fourth pass of
// 64 x kBoundSlots lists each and keep their k smallest keys; wavefront 0
// then merges the four sorted results (a key held by two of them is one row,
// counted once) up to the k-th.  With U known, the work-group certifies the
// query's items by it and lists the others for the rerank.
__global__ void __launch_bounds__(256) k_query_bound(StoreView s, QueryView qv, RoundBufs b, int64_t nq, int mq,
                                                     int kprime, int kmax, int cmax, float eps_max,
                                                     const uint64_t *__restrict__ cand, float *qbound) {
  extern __shared__ uint64_t bsm[];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  uint64_t *buf0 = bsm + static_cast<size_t>(wave) * 2 * kmax, *buf1 = buf0 + kmax;
  int *s_n = reinterpret_cast<int *>(bsm + 8 * static_cast<size_t>(kmax));  // [4] result sizes
  int *s_res = s_n + 4;                                                     // [4] result offsets
  float *s_u = reinterpret_cast<float *>(s_res + 4);                         // the query's bound
  // after a capacity overflow the item lists were never placed
  if (b.ctl[kCtlOverflow] != 0) return;
  const int N = s.N, m = s.m;
  constexpr int kPass = kWave * kBoundSlots;
  for (int64_t q = blockIdx.x; q < nq; q += gridDim.x) {
    const int n_it = b.qitem_cnt[q];
    const int k = b.kq[q];
    float U = fminf(b.tau[q], b.taud[q]);  // (taud only falls; the scan is over)
    if (n_it > 0) {
      const int nlists = n_it * cmax;
      uint64_t *in = buf0, *out = buf1;
      int n_in = 0;
      for (int l0 = wave * kPass; l0 < nlists; l0 += 4 * kPass) {
        const int nl = nlists - l0 < kPass ? nlists - l0 : kPass;
        n_in = bound_pass(q, N, k, kprime, mq, b.chunk, cmax, b, s, cand, l0, nl, in, n_in, out, lane);
        uint64_t *t = in;
        in = out;
        out = t;
      }
      if (lane == 0) {
        s_n[wave] = n_in;
        s_res[wave] = static_cast<int>(in - bsm);  // offset of this wavefront's result
      }
      __syncthreads();
      if (wave == 0) {
        // lanes 0..3 walk the four sorted results
        const int w = lane < 4 ? lane : 0;
        const uint64_t *res = bsm + s_res[w];
        const int cnt = lane < 4 ? s_n[w] : 0;
        int pos = 0;
        uint64_t hd = cnt > 0 ? res[0] : kKeyMax;
        uint64_t g = kKeyMax;
        int o = 0;
        while (o < k) {
          g = wave_min_u64(hd);
          if (g == kKeyMax) break;  // fewer than k keys in all
          ++o;
          if (hd == g) {
            ++pos;
            hd = pos < cnt ? res[pos] : kKeyMax;
          }
        }
        if (o == k) {
          // the key's distance was rounded down to its truncation step: the
          // computed value is at most the step's largest float
          const float kt = key_d2(g);
          const double kd = static_cast<double>(kt < __builtin_inff() ? u2f(f2u(kt) | ((1u << kDropBits) - 1)) : kt);
          const double v = sqrt(kd + bf16_delta(static_cast<double>(qv.qn16[q]), m)) + qv.qeps[q] + eps_max;
          float u = static_cast<float>(v);
          if (static_cast<double>(u) < v) u = nextafterf(u, __builtin_inff());
          U = u < U ? u : U;
        }
        if (lane == 0) *s_u = U;
      }
      __syncthreads();
      U = *s_u;
      // the query's items: certify by U what can be, list the rest in item_live
      for (int r0 = wave * kWave; r0 < n_it; r0 += 4 * kWave) {
        const int r = r0 + lane;
        const bool live = r < n_it && item_live_after_bound(s, qv, b, mq, kprime, cand, b.qitem_idx[q * N + r], q, U);
        const uint64_t mask = __ballot(live);
        if (mask != 0) {
          const int lead = __ffsll(static_cast<unsigned long long>(mask)) - 1;
          int at = 0;
          if (lane == lead)
            at = static_cast<int>(atomicAdd(reinterpret_cast<unsigned long long *>(b.ctl + kCtlLive),
                                            static_cast<unsigned long long>(__popcll(mask))));
          at = __shfl(at, lead, kWave);
          if (live) b.item_live[at + __popcll(mask & ((1ull << lane) - 1))] = b.qitem_idx[q * N + r];
        }
      }
    }
    if (threadIdx.x == 0) qbound[q] = U;
    __syncthreads();  // LDS is reused by the next query
  }
}

// Adds (q_t - x_t)^2 of four elements to the FP32 and the FP64 sum.
__device__ __forceinline__ void add_diff4(const float4 &a, const float4 &x, float &p, double &pd) {
  const float d0 = a.x - x.x, d1 = a.y - x.y, d2 = a.z - x.z, d3 = a.w - x.w;
  p = fmaf(d0, d0, p);
  p = fmaf(d1, d1, p);
  p = fmaf(d2, d2, p);
  p = fmaf(d3, d3, p);
  const double e0 = static_cast<double>(a.x) - static_cast<double>(x.x);
  const double e1 = static_cast<double>(a.y) - static_cast<double>(x.y);
  const double e2 = static_cast<double>(a.z) - static_cast<double>(x.z);
  const double e3 = static_cast<double>(a.w) - static_cast<double>(x.w);
  pd = fma(e0, e0, pd);
  pd = fma(e1, e1, pd);
  pd = fma(e2, e2, pd);
  pd = fma(e3, e3, pd);
}

// Sorts of the first n of 64 R keys by as few lanes as hold them.
template <int R, typename K>
__device__ __forceinline__ void sort_first(K (&v)[R], int n, int lane) {
  if (n <= 16 * R) wave_sort_regs<16>(v, lane);
  else wave_sort_regs<kWave>(v, lane);
}

// LDS of one wavefront of the rerank: the item's best keys (later its FP32
// keys), and their FP64 distances.
__host__ __device__ constexpr size_t rerank_slice_bytes(int R) { return static_cast<size_t>(64 * R) * 16; }

// One wavefront per item, up to 64 R candidates each (R registers per lane):
//  1. the item's kp best keys: its chunk lists are sorted, so each is merged
//     in registers into the best 64 R so far (7 to 9 comparator stages per
//     list), eight registers' worth of lists in flight together; in a search
//     round a list whose smallest key is beyond the query's bound U is
//     skipped whole;
//  2. the candidates that can still enter the query's top k (the keys are
//     ascending, so a prefix) have their rows read once, FP32 and FP64 sums
//     together, two groups of candidates in flight;
//  3. FP32 keys sorted for the k-th, whose error band names the exact
//     candidates; those sorted by (FP64 distance, row).
// Bound by latency (an item's loads are a chain of three), so the wavefront's
// LDS is kept to 16 bytes per candidate and the sorts off it.
template <int R>
__global__ void __launch_bounds__(256, 3) k_item_rerank(StoreView s, QueryView qv, RoundBufs b, int mq, int kprime,
                                                        int kmax, int bf16, const uint64_t *__restrict__ cand,
                                                        const float *__restrict__ qbound) {
  constexpr int kCap = kWave * R;
  __shared__ uint64_t smem[4 * 2 * kCap];
  const int wave = threadIdx.x / kWave, wpb = blockDim.x / kWave;
  uint64_t *keys = smem + static_cast<size_t>(wave) * 2 * kCap;  // [kCap]
  double *d64 = reinterpret_cast<double *>(keys + kCap);         // [kCap]
  const int lane = threadIdx.x & (kWave - 1);
  const int m = s.m;
  const int n_items = static_cast<int>(b.ctl[kCtlItems]);
  // the round's per-leaf item counts were consumed by its layout: zero them
  // for the merge, which counts rescan items into them
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < s.N;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    b.leaf_cnt[i] = 0;
  // error constants (see the certificate below)
  const double u = 1.0 / 16777216.0;  // 2^-24
  const float delta32 = static_cast<float>(2.0 * (m + 4) * u);
  // a search round reranks only the items k_query_bound listed
  const int n_work = qbound ? static_cast<int>(b.ctl[kCtlLive]) : n_items;
  for (int w_i = blockIdx.x * wpb + wave; w_i < n_work; w_i += gridDim.x * wpb) {
    const int item = __builtin_amdgcn_readfirstlane(qbound ? b.item_live[w_i] : w_i);
    const int L = b.item_leaf[item];
    const int64_t q = b.item_q[item];
    // everything else the item needs from memory, requested together
    const int k = b.kq[q];
    const int ist0 = b.leaf_istart[L], ist1 = b.leaf_istart[L + 1];
    const int64_t off0 = s.leaf_off[L], off1 = s.leaf_off[L + 1];
    const float tau_q = b.tau[q], qn_q = qv.qn16[q], qe_q = qv.qeps[q], le_L = s.leaf_eps[L];
    const float U = qbound ? qbound[q] : __builtin_inff();
    const int64_t t0 = b.tile_start[L];
    const int pos = item - ist0;
    const int g = pos / mq, j = pos - (pos / mq) * mq;
    const int C = static_cast<int>((off1 - off0 + b.chunk - 1) / b.chunk);
    const int G = (ist1 - ist0 + mq - 1) / mq;
    // the query's own candidate count (its lists hold kp keys in kprime slots)
    const int kp = item_kprime(b.kp_query, kprime, k, bf16 != 0);
    const int PKi = pow2_at_least(kp < 2 ? 2 : kp);
    const int n = C * kprime;
    const double dq = bf16_delta(static_cast<double>(qn_q), m);
    uint64_t best[R];  // key e in lane e / R, register e mod R
    if (kp <= kSelectMax && n <= kWave * kSelectPerLane) {
      // few keys wanted from many: kp rounds of a wavefront minimum, each
      // lane holding as few registers as n needs
      if (n <= kWave) select_keys<1>(cand, t0, G, g, mq, j, kprime, kp, n, lane, keys);
      else if (n <= 4 * kWave) select_keys<4>(cand, t0, G, g, mq, j, kprime, kp, n, lane, keys);
      else select_keys<kSelectPerLane>(cand, t0, G, g, mq, j, kprime, kp, n, lane, keys);
      wave_lds_sync();
#pragma unroll
      for (int r = 0; r < R; ++r) best[r] = lane * R + r < kp ? keys[lane * R + r] : kKeyMax;
    } else {
      // Search rounds: a key whose squared distance exceeds T (rounded up
      // past every key the exact test below keeps) has a lower bound above
      // U, and so have the keys after it in its list.  The smallest key
      // dropped this way also certifies every row its list left out.
      float T = __builtin_inff();
      if (U < __builtin_inff()) {
        const double t = static_cast<double>(U) + qe_q + le_L;
        T = static_cast<float>((t * t + dq) * (1.0 + 1e-6));
        T = nextafterf(T, __builtin_inff());
      }
      const uint32_t tb = f2u(T);
#pragma unroll
      for (int r = 0; r < R; ++r) best[r] = kKeyMax;
      constexpr int kLists = 8 / R;  // lists in flight together
      for (int c0 = 0; c0 < C; c0 += kLists) {
        uint64_t w[kLists][R];
#pragma unroll
        for (int v = 0; v < kLists; ++v)
#pragma unroll
          for (int r = 0; r < R; ++r) {
            // descending: lane 63's last register holds the list's smallest key
            const int e = kCap - 1 - (lane * R + r);
            const int c = c0 + v < C ? c0 + v : c0;
            const bool in = c0 + v < C && e < kp;
            const uint64_t x = cand[((t0 + static_cast<int64_t>(c) * G + g) * mq + j) * kprime + (e < kp ? e : 0)];
            w[v][r] = in ? x : kKeyMax;
          }
#pragma unroll
        for (int v = 0; v < kLists; ++v) {
          const uint32_t head =
              static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w[v][R - 1] >> 32), kWave - 1));
          if (head > tb) continue;  // uniform: beyond U, empty, or past the item's lists
          wave_merge_low(best, w[v], lane);
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (lane * R + r >= kp) best[r] = kKeyMax;
        keys[lane * R + r] = best[r];
      }
      wave_lds_sync();
    }
    const uint64_t kth = keys[kp - 1];
    // the real candidates among the first kp; in search rounds only those
    // that can still enter the query's top k (lower bound not above U)
    int nc = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      bool use = best[r] != kKeyMax;
      if (use && qbound) {
        const double v = static_cast<double>(key_d2(best[r])) - dq;
        const double lower = (v > 0.0 ? sqrt(v) : 0.0) - qe_q - le_L;
        use = !(lower > static_cast<double>(U));
      }
      nc += __popcll(__ballot(use));
    }
    // FP32 scan items: the candidates' keys already hold FP32
    // direct-difference values (same error bound), ascending; only those
    // within the band of the k-th need their rows
    float band = __builtin_inff();
    int nr = nc;  // candidates whose rows are read
    if (!bf16) {
      if (nc >= k) band = key_d2(keys[k - 1]) * (1.0f + 2.0f * delta32);
      nr = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) nr += __popcll(__ballot(lane * R + r < nc && key_d2(best[r]) <= band));
    }
    // direct differences: CB candidates at a time, GL lanes each, 4
    // consecutive elements per lane; two such groups in flight
    const float *qp = qv.q32 + q * m;
    const int CB = PKi < 8 ? PKi : 8, GL = kWave / CB;
    const int sub = lane & (GL - 1), cb = lane / GL;
    for (int e0 = 0; e0 < nr; e0 += 2 * CB) {
      const int ea = e0 + cb, eb = e0 + CB + cb;
      const bool two = e0 + CB < nr;  // uniform
      const uint32_t ra = key_row(keys[ea < nr ? ea : nr - 1]);
      const uint32_t rb = two ? key_row(keys[eb < nr ? eb : nr - 1]) : ra;
      const float *xa = s.x32 + static_cast<int64_t>(ra) * m, *xb = s.x32 + static_cast<int64_t>(rb) * m;
      float pa = 0.0f, pb = 0.0f;
      double da = 0.0, db = 0.0;
      if (two) {
#pragma unroll 4
        for (int t = 4 * sub; t < m; t += 4 * GL) {
          const float4 a = *reinterpret_cast<const float4 *>(qp + t);
          const float4 x = *reinterpret_cast<const float4 *>(xa + t);
          const float4 y = *reinterpret_cast<const float4 *>(xb + t);
          add_diff4(a, x, pa, da);
          add_diff4(a, y, pb, db);
        }
      } else {
#pragma unroll 8
        for (int t = 4 * sub; t < m; t += 4 * GL) {
          const float4 a = *reinterpret_cast<const float4 *>(qp + t);
          const float4 x = *reinterpret_cast<const float4 *>(xa + t);
          add_diff4(a, x, pa, da);
        }
      }
      for (int o = GL >> 1; o > 0; o >>= 1) {
        pa += __shfl_xor(pa, o, kWave);
        da += __shfl_xor(da, o, kWave);
      }
      if (two)
        for (int o = GL >> 1; o > 0; o >>= 1) {
          pb += __shfl_xor(pb, o, kWave);
          db += __shfl_xor(db, o, kWave);
        }
      wave_lds_sync();  // this step's rows are read before their keys are replaced
      if (sub == 0) {
        if (ea < nr) {
          if (bf16) keys[ea] = make_key(pa, ra);
          d64[ea] = da;
        }
        if (two && eb < nr) {
          if (bf16) keys[eb] = make_key(pb, rb);
          d64[eb] = db;
        }
      }
    }
    wave_lds_sync();
    uint64_t p32[R];
    ExactKey ex[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int e = lane * R + r;
      p32[r] = e < nr ? keys[e] : kKeyMax;
      ex[r].d = static_cast<uint64_t>(__double_as_longlong(e < nr ? d64[e] : __builtin_inf()));
      ex[r].row = e < nr ? key_row(p32[r]) : 0xffffffffu;
    }
    // FP64 for every candidate within the FP32 error band of the k-th
    int nb = nr;
    if (bf16) {
      if (nc >= k) {
        uint64_t srt[R];
#pragma unroll
        for (int r = 0; r < R; ++r) srt[r] = p32[r];
        if (nr > 1) sort_first<R>(srt, nr, lane);
        uint32_t kd = 0;
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (r == (k - 1) % R) kd = static_cast<uint32_t>(srt[r] >> 32);
        band = u2f(__builtin_amdgcn_readlane(kd, (k - 1) / R)) * (1.0f + 2.0f * delta32);
      }
      nb = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool inb = lane * R + r < nr && key_d2(p32[r]) <= band;
        if (!inb) {
          ex[r].d = static_cast<uint64_t>(__double_as_longlong(__builtin_inf()));
          ex[r].row = 0xffffffffu;
        }
        nb += __popcll(__ballot(inb));
      }
    }
    if (nr > 1) sort_first<R>(ex, nr, lane);
    const int keep = nb < k ? nb : k;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int e = lane * R + r;
      if (e < keep) {
        b.item_d2[static_cast<int64_t>(item) * kmax + e] = __longlong_as_double(static_cast<long long>(ex[r].d));
        b.item_row[static_cast<int64_t>(item) * kmax + e] = static_cast<int32_t>(ex[r].row);
      }
    }
    // Certificate: every row of the item outside the candidate list has a
    // scan key >= kth.  BF16: the computed value is within delta16 of the
    // exact squared distance of the bf16 vectors, and rounding moved q and x
    // by at most qeps and leaf_eps, so d(q, x) >= sqrt(kth - delta16) - eps.
    // FP32: the direct-difference value is within a relative delta32.
    // With a tau threshold T (search rounds), rows at or above T were never
    // candidates, so the list's own bound is capped by T's.  (Rows of lists
    // skipped by U, and candidates past it, are farther than U, which is at
    // least the query's new tau.)
    if (lane == 0) {
      float bound = __builtin_inff();
      float kd = kth != kKeyMax ? key_d2(kth) : __builtin_inff();
      if (bf16 && b.use_tau) kd = fminf(kd, tau_threshold(tau_q, qn_q, qe_q, le_L, m));
      if (kd < __builtin_inff()) {
        if (bf16) {
          double v = static_cast<double>(kd) - dq;
          bound = static_cast<float>((v > 0.0 ? sqrt(v) : 0.0) - qe_q - le_L);
        } else {
          bound = static_cast<float>(sqrt(static_cast<double>(kd) * (1.0 - delta32)));
        }
      }
      b.item_cnt[item] = keep;
      b.item_bound[item] = bound;
    }
    wave_lds_sync();
  }
}

}  // namespace

void launch_query_bound(StoreView s, QueryView q, RoundBufs b, int64_t nq, int mq, int kprime, int kmax, int cmax,
                        float eps_max, const uint64_t *cand, float *qbound, hipStream_t st) {
  if (nq <= 0) return;
  const size_t lds = 4 * 2 * static_cast<size_t>(kmax) * sizeof(uint64_t) + 12 * sizeof(int);
  const int64_t blocks = nq;  // one work-group per query
  hipLaunchKernelGGL(k_query_bound, dim3(static_cast<unsigned>(blocks < 65536 ? blocks : 65536)), dim3(256), lds, st, s,
                     q, b, nq, mq, kprime, kmax, cmax, eps_max, cand, qbound);
  LAUNCH_OK("query_bound");
}

void launch_item_rerank(StoreView s, QueryView q, RoundBufs b, int mq, int kprime, int kmax, bool bf16,
                        const uint64_t *cand, int grid, hipStream_t st, const float *qbound) {
  const dim3 blocks(ceil_div(grid, 4));  // four items (wavefronts) per work-group
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, blocks, dim3(256), 0, st, s, q, b, mq, kprime, kmax, bf16 ? 1 : 0, cand, qbound);
  };
  if (kprime <= 64) launch(k_item_rerank<1>);
  else if (kprime <= 128) launch(k_item_rerank<2>);
  else launch(k_item_rerank<4>);
  LAUNCH_OK("item_rerank");
}

}  // namespace leafi
