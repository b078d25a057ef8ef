// Per-item rerank of a round's candidate lists and the per-query bound that
// lets a search round skip items and candidates (SearchNode of Algorithm 2:
// the result update after a leaf's scan).
//
// After a pass's scan every (query, tile) list holds its kprime best keys
// (truncated BF16 or FP32 squared distances with rows).  k_query_bound finds
// per query an upper bound U of its k-th distance after the round; items whose
// every candidate is provably beyond U are certified by it; k_item_rerank
// merges each other item's chunk lists
// and reranks its candidates in FP32 (FP64 within the error band of the k-th),
// writing the item's exact top-k and the bound that certifies the rest.
#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "kernels.h"
#include "scan_bounds.h"
#include "wave_sort.h"

namespace leafi {

namespace {

// Selection instead of a full sort when at most kSelectMax of at most
// 64 * kSelectPerLane chunk candidates are wanted.
constexpr int kSelectMax = kCandFill;
constexpr int kSelectPerLane = 16;

// The kp smallest of an item's n chunk-list keys (kprime slots per chunk)
// into buf (ascending, kKeyMax past the last real key): kp rounds of a
// wavefront minimum over the keys above the round before's (keys are unique),
// U per lane in registers (unconditional loads of clamped entries, so all of a
// lane's loads are in flight together; the first kp <= kCandFill slots of each
// list, n = lists x kp >= 1 in all, so entry 0 exists; n <= 64 U).
template <int U>
__device__ inline void select_keys(const uint64_t *__restrict__ cand, int64_t t0, int G, int g, int mq, int j,
                                   int kprime, int kp, int n, int lane, uint64_t *buf) {
  uint64_t mine[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = lane + u * kWave;
    const int ec = e < n ? e : 0;
    const int c = ec / kp;
    const uint64_t v = cand[((t0 + static_cast<int64_t>(c) * G + g) * mq + j) * kprime + (ec - c * kp)];
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
// by key (bf16 squared distance, row).  Any k of their keys belong to k
// distinct rows (a leaf is in a round once per query, and its chunks' rows
// are apart), each no farther than sqrt(key + delta16) + eps_q + eps_L, so the
// query's k-th exact distance after this round's merge is at most U =
// sqrt(kth smallest key + delta16) + eps_q + max_L eps_L (and at most its tau
// before the round).  A candidate whose lower bound sqrt(key - delta16) -
// eps_q - eps_L exceeds U can never enter the query's top k, so the rerank
// skips its FP32 and FP64 distances.

constexpr int kBoundKeys = 2048;  // keys collected per query (more would only tighten its bound)

// One work-group per query.  The scan has left a bound already (taud: the
// least k-th key of any one list, which for k = 1 is the smallest key of all:
// those queries have nothing to do here, and a batch of them skips the
// launch), so only the keys below it matter: each thread walks its lists'
// heads while they are, most stop at the first, and the k-th smallest of the
// few hundred collected distances is found bit by bit by one wavefront.
// 1,024 queries of k <= 100 over 10M series: 96 us by a tournament over the
// list heads, now 58; 4,096 of k <= 50 over 2,198 leaves: 206, now 156, mostly
// the lists' addresses.
__global__ void __launch_bounds__(256) k_query_bound(StoreView s, QueryView qv, RoundBufs b, int64_t nq, int mq,
                                                     int kprime, int cmax, float eps_max,
                                                     const uint64_t *__restrict__ cand) {
  __shared__ uint32_t buf[kBoundKeys];
  __shared__ int s_n;
  // after a capacity overflow the item lists were never placed
  if (b.ctl[kCtlOverflow] != 0) return;
  const int N = s.N, m = s.m;
  for (int64_t q = blockIdx.x; q < nq; q += gridDim.x) {
    const int n_it = b.qitem_cnt[q];
    const int k = b.kq[q];
    if (n_it <= 0 || k <= 1) continue;  // uniform
    const float U = fminf(b.tau[q], b.taud[q]);
    const double dq = bf16_delta(static_cast<double>(qv.qn16[q]), m);
    const float qe = qv.qeps[q];
    // keys from here on are not below the bound (a rounding either way only
    // adds or drops a key)
    uint32_t top = 0xffffffffu;
    if (U < __builtin_inff()) {
      const double t = static_cast<double>(U) - qe - eps_max;
      top = t > 0.0 ? f2u(static_cast<float>(fmax(t * t - dq, 0.0))) : 0u;
    }
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const int kp = item_kprime(b.kp_query, kprime, k, true);
    const int nlists = n_it * cmax;
    for (int lam = threadIdx.x; lam < nlists; lam += 256) {
      const int r = lam / cmax, c = lam - r * cmax;
      const int idx = b.qitem_idx[q * N + r];
      const int L = b.item_leaf[idx];
      const int ist0 = b.leaf_istart[L], ist1 = b.leaf_istart[L + 1];
      const int C = static_cast<int>((s.leaf_off[L + 1] - s.leaf_off[L] + b.chunk - 1) / b.chunk);
      if (c >= C) continue;
      const int p = idx - ist0, g = p / mq, j = p - g * mq, G = (ist1 - ist0 + mq - 1) / mq;
      const uint64_t *list = cand + (tile_of(b.tile_start, L, g, c, G) * mq + j) * kprime;
      constexpr int kStep = 4;  // keys in flight together
      for (int e0 = 0; e0 < kp; e0 += kStep) {
        uint32_t v[kStep];
#pragma unroll
        for (int u = 0; u < kStep; ++u) v[u] = static_cast<uint32_t>(list[e0 + u < kp ? e0 + u : kp - 1] >> 32);
        int n = 0;
        bool below = true;  // (past the list's end its slots hold anything)
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
          below = below && e0 + u < kp && v[u] < top && v[u] < f2u(__builtin_inff());
          n += below ? 1 : 0;
        }
        if (n == 0) break;
        const int at = __hip_atomic_fetch_add(&s_n, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
        for (int u = 0; u < kStep; ++u)
          if (u < n && at + u < kBoundKeys) buf[at + u] = v[u];  // the list is sorted: its first n
        if (n < kStep || at >= kBoundKeys) break;
      }
    }
    __syncthreads();
    const int n = s_n < kBoundKeys ? s_n : kBoundKeys;
    if (n >= k && threadIdx.x < kWave) {
      const int lane = threadIdx.x;
      uint32_t kth = 0;  // the largest value with fewer than k keys below it
      auto select = [&](auto regs) {
        constexpr int kR = decltype(regs)::value;
        uint32_t v[kR];
#pragma unroll
        for (int u = 0; u < kR; ++u) v[u] = lane + kWave * u < n ? buf[lane + kWave * u] : 0xffffffffu;
        for (int bit = 30; bit >= kDropBits; --bit) {
          const uint32_t test = kth | 1u << bit;
          int below = 0;
#pragma unroll
          for (int u = 0; u < kR; ++u) below += __popcll(__ballot(v[u] < test));
          if (below < k) kth = test;
        }
      };
      if (n <= 4 * kWave) select(std::integral_constant<int, 4>{});
      else if (n <= 12 * kWave) select(std::integral_constant<int, 12>{});
      else select(std::integral_constant<int, kBoundKeys / kWave>{});
      if (lane == 0) {
        // the key's distance was rounded down to its truncation step: the
        // computed value is at most the step's largest float
        const double kd = static_cast<double>(u2f(kth | ((1u << kDropBits) - 1)));
        const double v = sqrt(kd + dq) + qe + eps_max;
        float u = static_cast<float>(v);
        if (static_cast<double>(u) < v) u = nextafterf(u, __builtin_inff());
        if (u < b.taud[q]) b.taud[q] = u;
      }
    }
    __syncthreads();  // LDS is reused by the next query
  }
}

// One item of a search round: each chunk list is sorted, so its first key is
// its smallest, and every row of the item has a key at least the smallest of
// them (or was never a candidate: key >= the tau threshold).  When even that
// bound exceeds the query's bound U, no row of the item can enter the query's
// top k: the item contributes nothing and is certified by that bound (no
// sort, no rerank).  `sub` consecutive lanes (a power of two; this one the
// l-th of them) share the item's lists.  Returns whether the item still needs
// its rerank.
__device__ inline bool item_live_after_bound(const StoreView &s, const QueryView &qv, const RoundBufs &b, int mq,
                                             int kprime, const uint64_t *__restrict__ cand, int item, int l, int sub) {
  const int m = s.m;
  const int L = b.item_leaf[item];
  const int64_t q = b.item_q[item];
  const int ist0 = b.leaf_istart[L], ist1 = b.leaf_istart[L + 1];
  const int64_t off0 = s.leaf_off[L], off1 = s.leaf_off[L + 1];
  const float tau_q = b.tau[q], qn_q = qv.qn16[q], qe_q = qv.qeps[q], le_L = s.leaf_eps[L];
  const float U = fminf(tau_q, b.taud[q]);
  const int64_t t0 = b.tile_start[L];
  const int pos = item - ist0;
  const int g = pos / mq, j = pos - g * mq;
  const int C = static_cast<int>((off1 - off0 + b.chunk - 1) / b.chunk);
  const int G = (ist1 - ist0 + mq - 1) / mq;
  uint32_t h = 0xffffffffu;  // the distance bits of an empty list's keys
  for (int c = l; c < C; c += sub)
    h = min(h, static_cast<uint32_t>(cand[((t0 + static_cast<int64_t>(c) * G + g) * mq + j) * kprime] >> 32));
  for (int o = sub / 2; o > 0; o /= 2) h = min(h, static_cast<uint32_t>(__shfl_xor(static_cast<int>(h), o, kWave)));
  float kd = h != 0xffffffffu ? u2f(h) : __builtin_inff();
  kd = fminf(kd, tau_threshold(tau_q, qn_q, qe_q, le_L, m));
  double lower = -1.0;
  if (kd < __builtin_inff()) {
    const double v = static_cast<double>(kd) - bf16_delta(qn_q, m);
    lower = (v > 0.0 ? sqrt(v) : 0.0) - qe_q - le_L;
  }
  if (lower > static_cast<double>(U)) {
    if (l == 0) {
      float lb = static_cast<float>(lower);
      if (static_cast<double>(lb) > lower) lb = nextafterf(lb, -__builtin_inff());
      b.item_cnt[item] = 0;
      b.item_bound[item] = lb;
    }
    return false;
  }
  return true;
}

// The items of a search round that the bounds leave, listed in item_live
// (ctl[kCtlLive] of them).  One lane per item, neighbours in a leaf: they share
// most of what they read, and their counts and certificates are written in
// runs (3.1M items 141 us; tested by query instead 264).
__global__ void __launch_bounds__(256) k_item_live(StoreView s, QueryView qv, RoundBufs b, int mq, int kprime,
                                                   const uint64_t *__restrict__ cand) {
  __shared__ int s_at[4];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t n_items = b.ctl[kCtlItems];
  for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * 256; i0 < n_items; i0 += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t i = i0 + threadIdx.x;
    const int item = static_cast<int>(i);
    const bool live = i < n_items && item_live_after_bound(s, qv, b, mq, kprime, cand, item, 0, 1);
    const uint64_t mask = __ballot(live);
    if (lane == 0) s_at[wave] = __popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
      const int n = s_at[0] + s_at[1] + s_at[2] + s_at[3];
      int at = n ? static_cast<int>(atomicAdd(reinterpret_cast<unsigned long long *>(b.ctl + kCtlLive),
                                              static_cast<unsigned long long>(n)))
                 : 0;
      for (int w = 0; w < 4; ++w) {
        const int c = s_at[w];
        s_at[w] = at;
        at += c;
      }
    }
    __syncthreads();
    if (live) b.item_live[s_at[wave] + __popcll(mask & ((1ull << lane) - 1))] = item;
    __syncthreads();  // s_at is reused
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

// What a rerank's wavefronts work on: every item, every item after its test
// against its query's bound, or the items k_item_live listed.
enum RerankItems { kRerankAll, kRerankTest, kRerankListed };

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
                                                        RerankItems which) {
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
  const bool use_bound = which != kRerankAll;
  const int n_work = which == kRerankListed ? static_cast<int>(b.ctl[kCtlLive]) : n_items;
  const int n_waves = static_cast<int>(gridDim.x) * wpb;
  int per = 1;  // items a wavefront tests at a time, neighbours
  if (which == kRerankTest)
    while (per < kWave && static_cast<int64_t>(n_waves) * per * 8 <= n_items) per *= 2;
  const int sub = kWave / per, l0 = lane / sub * sub;  // lanes l0 .. l0 + sub share an item's test
  for (int64_t w_i = static_cast<int64_t>(blockIdx.x * wpb + wave) * per; w_i < n_work;
       w_i += static_cast<int64_t>(n_waves) * per) {
    uint64_t todo = 1;
    if (which == kRerankTest) {
      const int item = static_cast<int>(w_i) + lane / sub;
      const bool live = item < n_items && item_live_after_bound(s, qv, b, mq, kprime, cand, item, lane - l0, sub);
      todo = __ballot(live && lane == l0);
    }
    for (; todo != 0; todo &= todo - 1) {
      const int at = static_cast<int>(w_i) + __builtin_ctzll(todo) / sub;
      const int item = __builtin_amdgcn_readfirstlane(which == kRerankListed ? b.item_live[at] : at);
      const int L = b.item_leaf[item];
      const int64_t q = b.item_q[item];
      // everything else the item needs from memory, requested together
      const int k = b.kq[q];
      const int ist0 = b.leaf_istart[L], ist1 = b.leaf_istart[L + 1];
      const int64_t off0 = s.leaf_off[L], off1 = s.leaf_off[L + 1];
      const float tau_q = b.tau[q], qn_q = qv.qn16[q], qe_q = qv.qeps[q], le_L = s.leaf_eps[L];
      const float U = use_bound ? fminf(tau_q, b.taud[q]) : __builtin_inff();
      const int64_t t0 = b.tile_start[L];
      const int pos = item - ist0;
      const int g = pos / mq, j = pos - (pos / mq) * mq;
      const int C = static_cast<int>((off1 - off0 + b.chunk - 1) / b.chunk);
      const int G = (ist1 - ist0 + mq - 1) / mq;
      // the query's own candidate count (its lists hold kp keys in kprime slots)
      const int kp = item_kprime(b.kp_query, kprime, k, bf16 != 0);
      const int PKi = pow2_at_least(kp < 2 ? 2 : kp);
      const int n = C * kp;
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
            // nothing past a list's end: a slot is before it if neither it
            // nor any lower slot (a higher register or lane) holds kKeyMax
            bool end = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const int e = kCap - 1 - (lane * R + r);
              end |= e < kp && w[v][r] == kKeyMax;
            }
            const uint64_t ends = __ballot(end);
            bool past = lane < kWave - 1 && (ends >> (lane + 1)) != 0;
#pragma unroll
            for (int r = R - 1; r >= 0; --r) {
              const int e = kCap - 1 - (lane * R + r);
              past |= e < kp && w[v][r] == kKeyMax;
              if (past) w[v][r] = kKeyMax;
            }
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
      // the real candidates among the first kp (not those at no finite
      // distance: their series are not finite); in search rounds only those
      // that can still enter the query's top k (lower bound not above U)
      int nc = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        bool use = static_cast<uint32_t>(best[r] >> 32) < f2u(__builtin_inff());
        if (use && use_bound) {
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
}

}  // namespace

void launch_query_bound(StoreView s, QueryView q, RoundBufs b, int64_t nq, int mq, int kprime, int kmax, int cmax,
                        float eps_max, const uint64_t *cand, hipStream_t st) {
  if (nq <= 0 || kmax <= 1) return;  // the scan's own bound is already the smallest key's
  // one work-group per query
  hipLaunchKernelGGL(k_query_bound, dim3(static_cast<unsigned>(nq < 65536 ? nq : 65536)), dim3(256), 0, st, s, q, b, nq,
                     mq, kprime, cmax, eps_max, cand);
  LAUNCH_OK("query_bound");
}

void launch_item_rerank(StoreView s, QueryView q, RoundBufs b, int mq, int kprime, int kmax, bool bf16,
                        const uint64_t *cand, int64_t items_bound, int grid, hipStream_t st, bool use_bound) {
  // Where the items' test against the bound goes: in the rerank itself for a
  // round that gives each wavefront at most one item, or of k = 1, whose few
  // items left take the same time; else in a launch of its own that lists the
  // items left, so that they spread evenly over the wavefronts.  (k = 1, 1,000
  // queries: 12 us, with the list 23.  k <= 10, one query: 15 and 19.  k <=
  // 100, 1,024 queries: 142, with the list 107.)
  const dim3 blocks(ceil_div(grid, 4));  // four items (wavefronts) per work-group
  const RerankItems which = !use_bound ? kRerankAll : kmax == 1 || items_bound <= grid ? kRerankTest : kRerankListed;
  if (which == kRerankListed) {
    const int64_t want = ceil_div(items_bound, 256), most = static_cast<int64_t>(device_cus()) * 32;
    hipLaunchKernelGGL(k_item_live, dim3(static_cast<unsigned>(want < most ? want : most)), dim3(256), 0, st, s, q, b,
                       mq, kprime, cand);
    LAUNCH_OK("item_live");
  }
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, blocks, dim3(256), 0, st, s, q, b, mq, kprime, kmax, bf16 ? 1 : 0, cand, which);
  };
  if (kprime <= 64) launch(k_item_rerank<1>);
  else if (kprime <= 128) launch(k_item_rerank<2>);
  else launch(k_item_rerank<4>);
  LAUNCH_OK("item_rerank");
}

}  // namespace leafi
