// Device build of the binary trees (median and midpoint splits): the same
// tree as build_tree's, node for node, from the summaries where they lie.
//
// All nodes of a level over capacity are split together.  The members stand
// in one array, grouped by node in depth-first order and ascending within a
// node, so a level is: each node's range of every (segment, statistic), the
// widest of them, the members' keys on it, the split point (midpoint, or the
// ceil(n/2)-th by (value, position): a radix select of the key's four bytes,
// then so many of its equals), and a stable partition of every node's members
// in place, which leaves the array in depth-first order again.  Work is dealt
// in chunks of kTreeChunk members of one node.  What bounds it is the ranges'
// read of every summary row per level (128 MB of 1M series x 16 segments) and
// about 20 launches a level.  1M x 256, 128 leaves: 1.6 ms; on the host, with
// the summaries' copy and first touch, 145.
#include <algorithm>
#include <cmath>

#include "device_util.h"
#include "engine.h"
#include "kernels.h"

namespace leafi {

namespace {

constexpr int kTreeChunk = 2048;   // members per work-group
constexpr int kTreeThreads = 256;
constexpr int kTreePer = kTreeChunk / kTreeThreads;

struct TreeChunk {
  int32_t node, start, len;  // node (of this pass), first position, members
};
struct TreeNode {
  int32_t start, n;          // members [start, start + n)
  int32_t c0, nc;            // its chunks
};
struct TreeSplit {
  int32_t col;       // 2 segment + statistic
  uint32_t key;      // members with keys below it go left, and the first `equal` of its equals
  int32_t equal;
  int32_t rank;      // radix select: rank still sought among the keys that share `key`'s bytes so far
  int32_t select;    // the select is on for this node
  int32_t left;      // members that go left
  float lo, hi;
};

// Floats as unsigned integers of the same order; -0 as +0, NaN last.
__device__ __host__ __forceinline__ uint32_t tree_key(float v) {
  union { float f; uint32_t u; } x;
  x.f = v;
  if (v != v) return 0xffffffffu;
  if (v == 0.0f) x.u = 0u;
  return x.u & 0x80000000u ? ~x.u : x.u | 0x80000000u;
}
__device__ __host__ __forceinline__ float tree_value(uint32_t k) {
  union { uint32_t u; float f; } x;
  x.u = k & 0x80000000u ? k & 0x7fffffffu : ~k;
  return x.f;
}
constexpr uint32_t kKeyPosInf = 0xff800000u, kKeyNegInf = 0x007fffffu;

__global__ void k_tree_iota(int32_t *ids, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) ids[i] = static_cast<int32_t>(i);
}

// Ranges of every column [nodes][2 S][2] start empty (the largest least and
// the least largest), the select's histograms at zero.
__global__ void k_tree_clear(uint32_t *rng, int64_t n_rng, uint32_t *hist, int64_t n_hist) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n_rng || i < n_hist;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    if (i < n_rng) rng[i] = i & 1 ? kKeyNegInf : kKeyPosInf;
    if (i < n_hist) hist[i] = 0;
  }
}

// Ranges of a chunk's members: G lanes (a power of two >= S) read one
// member's row, each keeping its columns' least and largest.
__global__ void __launch_bounds__(kTreeThreads) k_tree_ranges(const TreeChunk *__restrict__ chunks,
                                                              const int32_t *__restrict__ ids,
                                                              const float *__restrict__ mu, const float *__restrict__ sd,
                                                              int S, int G, uint32_t *rng) {
  __shared__ uint32_t red[kTreeThreads / kWave][4 * 64];
  const TreeChunk ch = chunks[blockIdx.x];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int s = lane % G, per = kWave / G;
  uint32_t v[4] = {kKeyPosInf, kKeyNegInf, kKeyPosInf, kKeyNegInf};
  if (s < S) {
#pragma unroll 4
    for (int i = wave * per + lane / G; i < ch.len; i += (kTreeThreads / kWave) * per) {
      const int64_t row = static_cast<int64_t>(ids[ch.start + i]) * S + s;
      const float a = mu[row], b = sd[row];
      if (a == a) {
        v[0] = min(v[0], tree_key(a));
        v[1] = max(v[1], tree_key(a));
      }
      if (b == b) {
        v[2] = min(v[2], tree_key(b));
        v[3] = max(v[3], tree_key(b));
      }
    }
  }
  for (int o = G; o < kWave; o *= 2) {
    v[0] = min(v[0], static_cast<uint32_t>(__shfl_xor(static_cast<int>(v[0]), o, kWave)));
    v[1] = max(v[1], static_cast<uint32_t>(__shfl_xor(static_cast<int>(v[1]), o, kWave)));
    v[2] = min(v[2], static_cast<uint32_t>(__shfl_xor(static_cast<int>(v[2]), o, kWave)));
    v[3] = max(v[3], static_cast<uint32_t>(__shfl_xor(static_cast<int>(v[3]), o, kWave)));
  }
  if (lane < S)
    for (int e = 0; e < 4; ++e) red[wave][4 * lane + e] = v[e];
  __syncthreads();
  // entry 4 s + 2 statistic + (0 least, 1 largest)
  for (int e = threadIdx.x; e < 4 * S; e += kTreeThreads) {
    uint32_t x = red[0][e];
    for (int w = 1; w < kTreeThreads / kWave; ++w) x = e & 1 ? max(x, red[w][e]) : min(x, red[w][e]);
    uint32_t *to = rng + static_cast<int64_t>(ch.node) * 4 * S + e;
    if (e & 1) atomicMax(to, x);
    else atomicMin(to, x);
  }
}

// One wavefront per node: the column of the largest seg_len x range^2 (ties:
// the lowest) and, for midpoint splits, its midpoint as a key.
__global__ void __launch_bounds__(kWave) k_tree_choose(const TreeNode *__restrict__ nodes,
                                                       const uint32_t *__restrict__ rng, int S, int m, int rule,
                                                       TreeSplit *split) {
  const int lane = threadIdx.x, node = blockIdx.x;
  const uint32_t *r = rng + static_cast<int64_t>(node) * 4 * S;
  double best = -1.0;
  int col = 0x7fffffff;
  for (int p = lane; p < 2 * S; p += kWave) {
    const int s = p / 2;
    const double len = static_cast<double>(((s + 1) * m) / S - (s * m) / S);
    const double d = static_cast<double>(tree_value(r[2 * p + 1])) - static_cast<double>(tree_value(r[2 * p]));
    const double score = len * (d * d);
    if (score > best) {
      best = score;
      col = p;
    }
  }
  for (int o = 1; o < kWave; o *= 2) {
    const double b2 = __shfl_xor(best, o, kWave);
    const int c2 = __shfl_xor(col, o, kWave);
    if (b2 > best || (b2 == best && c2 < col)) {
      best = b2;
      col = c2;
    }
  }
  if (lane != 0) return;
  TreeSplit t{};
  const bool any = col != 0x7fffffff;  // no column with a score: the first, its range taken as 0
  t.col = any ? col : 0;
  t.lo = any ? tree_value(r[2 * col]) : 0.0f;
  t.hi = any ? tree_value(r[2 * col + 1]) : 0.0f;
  if (rule == 1) {
    // the largest float not above lo + (hi - lo) / 2: members up to it go left
    const double mid = static_cast<double>(t.lo) + (static_cast<double>(t.hi) - static_cast<double>(t.lo)) / 2.0;
    float f = static_cast<float>(mid);
    if (static_cast<double>(f) > mid) f = nextafterf(f, -__builtin_inff());
    t.key = mid == mid ? tree_key(f) : 0u;
    t.equal = 0x7fffffff;
  } else {
    t.select = 1;
    t.rank = (nodes[node].n + 1) / 2 - 1;
  }
  split[node] = t;
}

// The members' keys on their node's column; midpoint splits count their left side.
__global__ void __launch_bounds__(kTreeThreads) k_tree_keys(const TreeChunk *__restrict__ chunks,
                                                            const int32_t *__restrict__ ids,
                                                            const float *__restrict__ mu, const float *__restrict__ sd,
                                                            int S, int rule, TreeSplit *split, uint32_t *keys) {
  __shared__ int s_n;
  const TreeChunk ch = chunks[blockIdx.x];
  const int col = split[ch.node].col;
  const uint32_t key = split[ch.node].key;
  const float *src = (col & 1 ? sd : mu) + col / 2;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  int n = 0;
#pragma unroll
  for (int u = 0; u < kTreePer; ++u) {
    const int i = threadIdx.x + u * kTreeThreads;
    if (i < ch.len) {
      const uint32_t k = tree_key(src[static_cast<int64_t>(ids[ch.start + i]) * S]);
      keys[ch.start + i] = k;
      n += k <= key ? 1 : 0;
    }
  }
  if (rule != 1) return;
  n = wave_sum(n);
  if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&s_n, n);
  __syncthreads();
  if (threadIdx.x == 0 && s_n > 0) atomicAdd(&split[ch.node].left, s_n);
}

// Midpoint splits with an empty side fall back to the median.
__global__ void k_tree_fallback(const TreeNode *__restrict__ nodes, int n_nodes, TreeSplit *split) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_nodes) return;
  TreeSplit &t = split[i];
  if (t.left > 0 && t.left < nodes[i].n) return;
  t.key = 0;
  t.equal = 0;
  t.select = 1;
  t.rank = (nodes[i].n + 1) / 2 - 1;
}

// One byte of the select: the histogram of the byte at `shift` over the keys
// that share the bytes found so far.
__global__ void __launch_bounds__(kTreeThreads) k_tree_hist(const TreeChunk *__restrict__ chunks,
                                                            const uint32_t *__restrict__ keys,
                                                            const TreeSplit *__restrict__ split, int shift,
                                                            uint32_t *hist) {
  __shared__ uint32_t h[256];
  const TreeChunk ch = chunks[blockIdx.x];
  if (!split[ch.node].select) return;  // uniform
  const uint32_t key = split[ch.node].key;
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t mask = shift == 24 ? 0u : ~0u << (shift + 8);
#pragma unroll
  for (int u = 0; u < kTreePer; ++u) {
    const int i = threadIdx.x + u * kTreeThreads;
    if (i < ch.len) {
      const uint32_t k = keys[ch.start + i];
      if (((k ^ key) & mask) == 0) atomicAdd(h + ((k >> shift) & 255u), 1u);
    }
  }
  __syncthreads();
  const uint32_t c = h[threadIdx.x];
  if (c) atomicAdd(hist + static_cast<int64_t>(ch.node) * 256 + threadIdx.x, c);
}

// One work-group of 256 per node: the byte whose bin holds the rank sought.
// After the last one `key` is the pivot and rank + 1 of its equals go left.
__global__ void __launch_bounds__(256) k_tree_pick(TreeSplit *split, int shift, uint32_t *hist) {
  __shared__ int32_t sh[4];
  const int node = blockIdx.x;
  TreeSplit &t = split[node];
  if (!t.select) return;  // uniform
  const int rank = t.rank;
  uint32_t *h = hist + static_cast<int64_t>(node) * 256 + threadIdx.x;
  const int32_t c = static_cast<int32_t>(*h);
  *h = 0;
  int32_t total;
  const int32_t before = block_scan_excl<256>(c, sh, total);
  __syncthreads();  // every thread has read the rank
  if (before <= rank && rank < before + c) {
    t.key |= static_cast<uint32_t>(threadIdx.x) << shift;
    t.rank = rank - before;
    if (shift == 0) t.equal = rank - before + 1;
  }
}

// A chunk's members below the split key and equal to it.
__global__ void __launch_bounds__(kTreeThreads) k_tree_count(const TreeChunk *__restrict__ chunks,
                                                             const uint32_t *__restrict__ keys,
                                                             const TreeSplit *__restrict__ split, int2 *cnt) {
  __shared__ int s_n[2];
  const TreeChunk ch = chunks[blockIdx.x];
  const uint32_t key = split[ch.node].key;
  if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
  __syncthreads();
  int lt = 0, eq = 0;
#pragma unroll
  for (int u = 0; u < kTreePer; ++u) {
    const int i = threadIdx.x + u * kTreeThreads;
    if (i < ch.len) {
      const uint32_t k = keys[ch.start + i];
      lt += k < key ? 1 : 0;
      eq += k == key ? 1 : 0;
    }
  }
  lt = wave_sum(lt);
  eq = wave_sum(eq);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    atomicAdd(s_n, lt);
    atomicAdd(s_n + 1, eq);
  }
  __syncthreads();
  if (threadIdx.x == 0) cnt[blockIdx.x] = make_int2(s_n[0], s_n[1]);
}

// One work-group per node: its chunks' counts become the counts before each.
__global__ void __launch_bounds__(256) k_tree_scan(const TreeNode *__restrict__ nodes, TreeSplit *split, int2 *cnt) {
  __shared__ int64_t sh[4];
  const TreeNode nd = nodes[blockIdx.x];
  int64_t run = 0;  // below in the low half, equal in the high half
  for (int b0 = 0; b0 < nd.nc; b0 += 256) {
    const int b = b0 + static_cast<int>(threadIdx.x);
    int2 c = make_int2(0, 0);
    if (b < nd.nc) c = cnt[nd.c0 + b];
    int64_t total;
    const int64_t x = run + block_scan_excl<256>(static_cast<int64_t>(c.x) + (static_cast<int64_t>(c.y) << 32), sh, total);
    if (b < nd.nc) cnt[nd.c0 + b] = make_int2(static_cast<int>(x & 0xffffffffll), static_cast<int>(x >> 32));
    run += total;
  }
  if (threadIdx.x == 0) {
    const int lt = static_cast<int>(run & 0xffffffffll), eq = static_cast<int>(run >> 32);
    split[blockIdx.x].left = lt + min(eq, split[blockIdx.x].equal);
  }
}

// The stable partition: thread t places the chunk's members 8 t .. 8 t + 7.
__global__ void __launch_bounds__(kTreeThreads) k_tree_scatter(const TreeChunk *__restrict__ chunks,
                                                               const TreeNode *__restrict__ nodes,
                                                               const TreeSplit *__restrict__ split,
                                                               const int2 *__restrict__ cnt,
                                                               const uint32_t *__restrict__ keys,
                                                               const int32_t *__restrict__ ids, int32_t *out) {
  __shared__ int32_t sh[kTreeThreads / kWave];
  const TreeChunk ch = chunks[blockIdx.x];
  const TreeNode nd = nodes[ch.node];
  const TreeSplit t = split[ch.node];
  const int2 base = cnt[blockIdx.x];
  int32_t id[kTreePer], c = 0;
  uint32_t k[kTreePer];
#pragma unroll
  for (int u = 0; u < kTreePer; ++u) {
    const int i = threadIdx.x * kTreePer + u;
    k[u] = i < ch.len ? keys[ch.start + i] : 0xffffffffu;
    id[u] = i < ch.len ? ids[ch.start + i] : 0;
    // below + (equal << 16): at most 2,048 of each in a chunk
    if (i < ch.len) c += k[u] < t.key ? 1 : k[u] == t.key ? 1 << 16 : 0;
  }
  int32_t total;
  const int32_t before = block_scan_excl<kTreeThreads>(c, sh, total);
  int lt = base.x + (before & 0xffff), eq = base.y + (before >> 16);
#pragma unroll
  for (int u = 0; u < kTreePer; ++u) {
    const int i = threadIdx.x * kTreePer + u;
    if (i < ch.len) {
      const bool below = k[u] < t.key, same = k[u] == t.key;
      const int left = lt + min(eq, t.equal);  // left members before this one
      const bool go = below || (same && eq < t.equal);
      const int at = ch.start - nd.start + i;  // its place in the node
      out[nd.start + (go ? left : t.left + at - left)] = id[u];
      lt += below ? 1 : 0;
      eq += same ? 1 : 0;
    }
  }
}

__global__ void __launch_bounds__(kTreeThreads) k_tree_copy(const TreeChunk *__restrict__ chunks,
                                                            const int32_t *__restrict__ from, int32_t *to) {
  const TreeChunk ch = chunks[blockIdx.x];
#pragma unroll
  for (int u = 0; u < kTreePer; ++u) {
    const int i = threadIdx.x + u * kTreeThreads;
    if (i < ch.len) to[ch.start + i] = from[ch.start + i];
  }
}

// Store rows from the tree: row off[L] + i of leaf L is its member i, the
// padding rows -1; and the members as 64-bit ids in tree order.
__global__ void __launch_bounds__(256) k_tree_rows(int64_t rows, int N, const int64_t *__restrict__ off,
                                                   const int64_t *__restrict__ first, const int32_t *__restrict__ ids,
                                                   int64_t *src, int32_t *leaf, int64_t *members) {
  const int64_t r = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (r >= rows) return;
  int lo = 0, hi = N;  // off[lo] <= r < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (off[mid] <= r) lo = mid;
    else hi = mid;
  }
  const int64_t at = first[lo] + r - off[lo];
  const bool real = at < first[lo + 1];
  const int64_t id = real ? ids[at] : -1;
  src[r] = id;
  leaf[r] = lo;
  if (real) members[at] = id;
}

// A pass's nodes and their chunks on the device.
struct TreePass {
  std::vector<TreeNode> nodes;
  std::vector<TreeChunk> chunks;
  void add(int64_t start, int64_t n) {
    TreeNode nd{static_cast<int32_t>(start), static_cast<int32_t>(n), static_cast<int32_t>(chunks.size()), 0};
    for (int64_t a = 0; a < n; a += kTreeChunk)
      chunks.push_back({static_cast<int32_t>(nodes.size()), static_cast<int32_t>(start + a),
                        static_cast<int32_t>(std::min<int64_t>(kTreeChunk, n - a))});
    nd.nc = static_cast<int32_t>(chunks.size()) - nd.c0;
    nodes.push_back(nd);
  }
};

}  // namespace

void device_tree(const float *mu, const float *sd, int64_t n, int S, int m, int capacity, int rule, int max_leaves,
                 DevBuf<int32_t> &ids, std::vector<int64_t> &sizes, std::vector<float> &boxes, hipStream_t st) {
  ids.alloc(n);
  DevBuf<int32_t> tmp(n);
  DevBuf<uint32_t> keys(n), rng, hist;
  DevBuf<TreeChunk> dchunks;
  DevBuf<TreeNode> dnodes;
  DevBuf<TreeSplit> dsplit;
  DevBuf<int2> dcnt;
  int G = 1;
  while (G < S) G *= 2;
  hipLaunchKernelGGL(k_tree_iota, dim3(static_cast<unsigned>(ceil_div(n, 256))), dim3(256), 0, st, ids.get(), n);
  LAUNCH_OK("tree_iota");
  auto ranges = [&](const TreePass &p, int64_t n_hist) {
    const int64_t n_rng = static_cast<int64_t>(p.nodes.size()) * 4 * S;
    rng.reserve(n_rng);
    dchunks.reserve(p.chunks.size());
    h2d(dchunks.get(), p.chunks.data(), p.chunks.size(), st);
    hipLaunchKernelGGL(k_tree_clear, dim3(static_cast<unsigned>(std::min<int64_t>(ceil_div(std::max(n_rng, n_hist), 256), 1024))),
                       dim3(256), 0, st, rng.get(), n_rng, hist.get(), n_hist);
    hipLaunchKernelGGL(k_tree_ranges, dim3(static_cast<unsigned>(p.chunks.size())), dim3(kTreeThreads), 0, st,
                       dchunks.get(), ids.get(), mu, sd, S, G, rng.get());
    LAUNCH_OK("tree_ranges");
  };
  std::vector<int64_t> all{n};  // the nodes in depth-first order, leaves so far and nodes still to split
  std::vector<TreeSplit> split;
  for (;;) {
    TreePass p;
    int64_t at = 0;
    for (int64_t c : all) {
      if (c > capacity) p.add(at, c);
      at += c;
    }
    if (p.nodes.empty() || static_cast<int>(all.size()) > max_leaves) break;
    const unsigned nn = static_cast<unsigned>(p.nodes.size()), nc = static_cast<unsigned>(p.chunks.size());
    dnodes.reserve(nn);
    dsplit.reserve(nn);
    dcnt.reserve(nc);
    hist.reserve(static_cast<size_t>(nn) * 256);
    h2d(dnodes.get(), p.nodes.data(), nn, st);
    ranges(p, static_cast<int64_t>(nn) * 256);
    hipLaunchKernelGGL(k_tree_choose, dim3(nn), dim3(kWave), 0, st, dnodes.get(), rng.get(), S, m, rule, dsplit.get());
    hipLaunchKernelGGL(k_tree_keys, dim3(nc), dim3(kTreeThreads), 0, st, dchunks.get(), ids.get(), mu, sd, S, rule,
                       dsplit.get(), keys.get());
    if (rule == 1)
      hipLaunchKernelGGL(k_tree_fallback, dim3(static_cast<unsigned>(ceil_div(nn, 256))), dim3(256), 0, st, dnodes.get(),
                         static_cast<int>(nn), dsplit.get());
    for (int shift = 24; shift >= 0; shift -= 8) {
      hipLaunchKernelGGL(k_tree_hist, dim3(nc), dim3(kTreeThreads), 0, st, dchunks.get(), keys.get(), dsplit.get(), shift,
                         hist.get());
      hipLaunchKernelGGL(k_tree_pick, dim3(nn), dim3(256), 0, st, dsplit.get(), shift, hist.get());
    }
    hipLaunchKernelGGL(k_tree_count, dim3(nc), dim3(kTreeThreads), 0, st, dchunks.get(), keys.get(), dsplit.get(),
                       dcnt.get());
    hipLaunchKernelGGL(k_tree_scan, dim3(nn), dim3(256), 0, st, dnodes.get(), dsplit.get(), dcnt.get());
    hipLaunchKernelGGL(k_tree_scatter, dim3(nc), dim3(kTreeThreads), 0, st, dchunks.get(), dnodes.get(), dsplit.get(),
                       dcnt.get(), keys.get(), ids.get(), tmp.get());
    hipLaunchKernelGGL(k_tree_copy, dim3(nc), dim3(kTreeThreads), 0, st, dchunks.get(), tmp.get(), ids.get());
    LAUNCH_OK("tree_split");
    split.resize(nn);
    d2h(split.data(), dsplit.get(), nn, st);
    HIP_OK(hipStreamSynchronize(st));
    std::vector<int64_t> next;
    next.reserve(all.size() + nn);
    size_t k = 0;
    for (int64_t c : all) {
      if (c > capacity) {
        const int64_t left = split[k++].left;
        if (left <= 0 || left >= c) fail(LEAFI_EINTERNAL, "device_tree: a split left one side empty");
        next.push_back(left);
        next.push_back(c - left);
      } else {
        next.push_back(c);
      }
    }
    all.swap(next);
  }
  sizes = std::move(all);
  if (static_cast<int>(sizes.size()) > max_leaves) return;  // the caller refuses it
  // the leaves' boxes: their ranges widened by one ulp
  TreePass p;
  int64_t at = 0;
  for (int64_t c : sizes) {
    p.add(at, c);
    at += c;
  }
  ranges(p, 0);
  std::vector<uint32_t> r(p.nodes.size() * 4 * static_cast<size_t>(S));
  d2h(r.data(), rng.get(), r.size(), st);
  HIP_OK(hipStreamSynchronize(st));
  boxes.resize(r.size());
  for (size_t i = 0; i < r.size(); ++i) boxes[i] = std::nextafter(tree_value(r[i]), i & 1 ? INFINITY : -INFINITY);
}

void launch_tree_rows(int64_t rows, int N, const int64_t *off, const int64_t *first, const int32_t *ids, int64_t *src,
                      int32_t *leaf, int64_t *members, hipStream_t st) {
  hipLaunchKernelGGL(k_tree_rows, dim3(static_cast<unsigned>(ceil_div(rows, 256))), dim3(256), 0, st, rows, N, off, first,
                     ids, src, leaf, members);
  LAUNCH_OK("tree_rows");
}

}  // namespace leafi
