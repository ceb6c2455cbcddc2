// Sorting by counting: a key's place is the number of keys before it.
#pragma once

#include "flix_device.hpp"

namespace flix {

constexpr u32 kRankKeys = 32;     // keys ranked by a workgroup of 256

template <typename K>
struct RankSmem {
  static constexpr u32 C = 16384 / sizeof(K);   // batch keys compared per round
  K k[C];
};

// Ranks of keys [32 unit, 32 unit + 32) among n keys (get(j): key j) in their
// stable order.  True in the lanes that hold one: key *i, *key, rank *at.  A
// wave holds eight keys in
// scalar registers and its lanes share the comparisons, so each batch key read
// from LDS serves eight (eight lanes per key, a read per comparison, left LDS
// the bound: 42 us for 16384 u64 keys, 31 so).  All 256 threads call.
template <typename K, typename F>
__device__ __forceinline__ bool rank_keys(F get, u32 n, u32 unit, RankSmem<K>& sm, u32* i, K* key,
                                          u32* at) {
  constexpr u32 C = RankSmem<K>::C, E = 16 / sizeof(K), Q = kRankKeys / 4;
  constexpr u32 G = 64 * E;   // keys a wave compares per step
  const u32 tid = threadIdx.x, lane = tid & 63u;
  const u32 i0 = unit * kRankKeys;
  const u32 iw = i0 + Q * (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  K x[Q];
  u32 rank[Q];
#pragma unroll
  for (u32 q = 0; q < Q; ++q) {
    x[q] = iw + q < n ? get(iw + q) : K(0);
    rank[q] = 0;
  }
  // a round's loads are all in flight at a time, the next round's while this
  // one is compared
  constexpr u32 L = C / 256;
  K buf[L];
  auto fetch = [&](u32 c0) {
#pragma unroll
    for (u32 r = 0; r < L; ++r) {
      const u32 j = c0 + r * 256 + tid;
      if (c0 + r * 256 < n) buf[r] = j < n ? get(j) : key_max<K>();
    }
  };
  fetch(0);
  for (u32 c0 = 0; c0 < n; c0 += C) {
    __syncthreads();   // the previous round's keys are compared
    const u32 cnt = n - c0 < C ? n - c0 : C;
    const u32 cpad = (cnt + G - 1) / G * G;
#pragma unroll
    for (u32 r = 0; r < L; ++r)
      if (r * 256 < cpad) sm.k[r * 256 + tid] = r * 256 < cnt ? buf[r] : key_max<K>();
    __syncthreads();
    if (c0 + C < n) fetch(c0 + C);
    // before this unit's keys equal keys count, after them they do not; among
    // them positions decide (the padding is after every key and below none)
    const u32 lo = i0 > c0 ? (i0 - c0 < cpad ? i0 - c0 : cpad) / G * G : 0u;
    const u32 last = i0 + kRankKeys > c0 ? (i0 + kRankKeys - c0 + G - 1) / G * G : 0u;
    const u32 mid = last > lo ? (last < cpad ? last : cpad) : lo;
    const u32 l0 = lane * E;
#pragma unroll 2
    for (u32 j = l0; j < lo; j += G) {
      const KeyVec<K, (int)E> v = *reinterpret_cast<const KeyVec<K, (int)E>*>(&sm.k[j]);
#pragma unroll
      for (u32 q = 0; q < Q; ++q)
#pragma unroll
        for (u32 e = 0; e < E; ++e) rank[q] += v.k[e] <= x[q] ? 1u : 0u;
    }
    for (u32 j = lo + l0; j < mid; j += G) {
      const KeyVec<K, (int)E> v = *reinterpret_cast<const KeyVec<K, (int)E>*>(&sm.k[j]);
#pragma unroll
      for (u32 q = 0; q < Q; ++q)
#pragma unroll
        for (u32 e = 0; e < E; ++e)
          rank[q] += (v.k[e] < x[q] || (v.k[e] == x[q] && c0 + j + e < iw + q)) ? 1u : 0u;
    }
#pragma unroll 2
    for (u32 j = mid + l0; j < cpad; j += G) {
      const KeyVec<K, (int)E> v = *reinterpret_cast<const KeyVec<K, (int)E>*>(&sm.k[j]);
#pragma unroll
      for (u32 q = 0; q < Q; ++q)
#pragma unroll
        for (u32 e = 0; e < E; ++e) rank[q] += v.k[e] < x[q] ? 1u : 0u;
    }
  }
  // lane q takes key q's rank
  u32 mine = 0;
  K xm = K(0);
#pragma unroll
  for (u32 q = 0; q < Q; ++q) {
    u32 r = rank[q];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) r += (u32)__shfl_xor((int)r, o, 64);
    if (lane == q) {
      mine = r;
      xm = x[q];
    }
  }
  *i = iw + lane;
  *key = xm;
  *at = mine;
  return lane < Q && iw + lane < n && mine < n;
}

}  // namespace flix
