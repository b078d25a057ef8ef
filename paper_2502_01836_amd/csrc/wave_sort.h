// Sorting and merging of keys held in the registers of one 64-lane wavefront.
//
// 64 R keys, R per lane; key i (in sorted order) sits in lane i / R, register
// i mod R.  The networks are bitonic in the form whose every comparator puts
// the smaller key at the lower index: each merge starts by comparing an index
// with its mirror in the block (lane xor 2^j - 1, register R - 1 - r), then
// halves.  All lane moves are VALU instructions (DPP within a 16-lane row,
// v_permlane16_swap / v_permlane32_swap across rows), so a stage neither
// touches LDS nor waits: what bounds a sort is its chain of 21 lane stages
// (about 4 instructions each per register), where the same network on LDS pays
// a round trip of over 100 cycles per stage.
#pragma once

#include "device_util.h"

namespace leafi {

// Exchanges the odd 16-lane rows of a with the even rows of b (gfx950).
__device__ __forceinline__ void permlane16_swap(uint32_t &a, uint32_t &b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
// Exchanges the upper 32 lanes of a with the lower 32 lanes of b (gfx950).
__device__ __forceinline__ void permlane32_swap(uint32_t &a, uint32_t &b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

template <int Ctrl>
__device__ __forceinline__ uint32_t dpp_all(uint32_t v) {
  return static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(static_cast<int>(v), static_cast<int>(v), Ctrl, 0xf, 0xf, false));
}

// v of lane (lane xor M), for the masks the networks use.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
  static_assert(M == 1 || M == 2 || M == 3 || M == 4 || M == 7 || M == 8 || M == 15 || M == 16 || M == 31 || M == 32 ||
                    M == 63,
                "xor mask");
  if constexpr (M == 1) return dpp_all<0xB1>(v);         // quad_perm 1,0,3,2
  else if constexpr (M == 2) return dpp_all<0x4E>(v);    // quad_perm 2,3,0,1
  else if constexpr (M == 3) return dpp_all<0x1B>(v);    // quad_perm 3,2,1,0
  else if constexpr (M == 4) return dpp_all<0x1B>(dpp_all<0x141>(v));
  else if constexpr (M == 7) return dpp_all<0x141>(v);   // row_half_mirror
  else if constexpr (M == 8) return dpp_all<0x128>(v);   // row_ror:8
  else if constexpr (M == 15) return dpp_all<0x140>(v);  // row_mirror
  else if constexpr (M == 16) {
    uint32_t a = v, b = v;
    permlane16_swap(a, b);  // a: the even rows' values in both rows of a pair, b: the odd rows'
    return (lane & 16) ? a : b;
  } else if constexpr (M == 31) return lane_xor<15>(lane_xor<16>(v, lane), lane);
  else if constexpr (M == 32) {
    uint32_t a = v, b = v;
    permlane32_swap(a, b);
    return (lane & 32) ? a : b;
  } else return lane_xor<31>(lane_xor<32>(v, lane), lane);
}
template <int M>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v, int lane) {
  const uint32_t lo = lane_xor<M>(static_cast<uint32_t>(v), lane);
  const uint32_t hi = lane_xor<M>(static_cast<uint32_t>(v >> 32), lane);
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// An FP64 squared distance's bits (non-negative doubles order like them),
// then a row.
struct ExactKey {
  uint64_t d;
  uint32_t row;
};
__device__ __forceinline__ bool operator<(const ExactKey &a, const ExactKey &b) {
  return a.d < b.d || (a.d == b.d && a.row < b.row);
}
template <int M>
__device__ __forceinline__ ExactKey lane_xor(const ExactKey &v, int lane) {
  return ExactKey{lane_xor<M>(v.d, lane), lane_xor<M>(v.row, lane)};
}

// c ? a : b, field by field (a select between two structs' addresses would
// put them in scratch memory).
template <typename K>
__device__ __forceinline__ K pick(bool c, const K &a, const K &b) {
  return c ? a : b;
}
__device__ __forceinline__ ExactKey pick(bool c, const ExactKey &a, const ExactKey &b) {
  return ExactKey{c ? a.d : b.d, c ? a.row : b.row};
}

template <typename K>
__device__ __forceinline__ void order_pair(K &lo, K &hi) {
  const bool le = lo < hi;
  const K a = pick(le, lo, hi), b = pick(le, hi, lo);
  lo = a;
  hi = b;
}
// The smaller of v and p on the low lane of a comparator, the larger on the high one.
template <typename K>
__device__ __forceinline__ K comparator(const K &v, const K &p, bool high) {
  return pick((v < p) != high, v, p);
}

// Comparators of lane stride S (registers pair with themselves), then every
// smaller stride, then the registers of a lane: finishes the merge of a
// bitonic sequence over 2 S lanes.
template <int S, typename K, int R>
__device__ __forceinline__ void halve(K (&v)[R], int lane) {
  if constexpr (S >= 1) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const K p = lane_xor<S>(v[r], lane);
      v[r] = comparator(v[r], p, (lane & S) != 0);
    }
    halve<S / 2>(v, lane);
  } else {
#pragma unroll
    for (int s = R / 2; s >= 1; s >>= 1)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if ((r & s) == 0) order_pair(v[r], v[r + s]);
  }
}

// Merges the two sorted halves of every block of 2 H lanes, and on.
template <int H, int L, typename K, int R>
__device__ __forceinline__ void merge_up(K (&v)[R], int lane) {
  if constexpr (2 * H <= L) {
    K p[R];
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = lane_xor<2 * H - 1>(v[R - 1 - r], lane);
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = comparator(v[r], p[r], (lane & H) != 0);
    halve<H / 2>(v, lane);
    merge_up<2 * H, L>(v, lane);
  }
}

// Ascending sort of the R L keys of every group of L lanes (L a power of two
// up to 64).
template <int L, typename K, int R>
__device__ __forceinline__ void wave_sort_regs(K (&v)[R], int lane) {
#pragma unroll
  for (int size = 2; size <= R; size <<= 1) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & (size / 2)) == 0) order_pair(v[r], v[(r / size) * size + size - 1 - r % size]);
#pragma unroll
    for (int s = size / 4; s >= 1; s >>= 1)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if ((r & s) == 0) order_pair(v[r], v[r + s]);
  }
  merge_up<1, L>(v, lane);
}

// The 64 R smallest keys of two sorted sets, sorted, into a: b holds the
// second set in descending order (lane, register mirrored).
template <typename K, int R>
__device__ __forceinline__ void wave_merge_low(K (&a)[R], const K (&b_desc)[R], int lane) {
#pragma unroll
  for (int r = 0; r < R; ++r) a[r] = pick(b_desc[r] < a[r], b_desc[r], a[r]);
  halve<32>(a, lane);
}

}  // namespace leafi
