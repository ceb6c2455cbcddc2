// Update batches too short to fill the chip: of their time the launches, the
// device-wide sort (a workgroup per top digit, few of them busy) and the pass
// over the whole directory were the most.  Here
//   rank_unit    sorts: every key counts the keys before it, compared with
//                the whole batch in LDS, and goes straight to its place (n^2
//                comparisons, spread over the chip, in one launch);
//   slice_unit   finds every key's bucket by the directory search of the
//                direct reads; the first key of each bucket becomes a work
//                item at its own position of a flat list, so nothing is
//                counted, claimed or cleared;
//   the apply kernels then take item i from position i (UpdArgs::flat).
// A slice unit leaves its part of the node bound in Ctl::part, which the apply
// kernels sum, so the bound needs no counter cleared beforehand; the sort clears
// the one counter that is left, of the workgroup-wide items.
#pragma once

#include "flix_direct.hpp"
#include "flix_update.hpp"

namespace flix {

// Longest batch of this form.  An insert, a delete and two lookups of n keys
// into 2^24, this form against the sort and the directory pass: n = 64 (u32)
// 50 against 106 us, 5000 72 against 100, 10000 99 against 110, 16384 127
// against 118 (u64: 131 against 132).  At 12288 the keys decide: an insert of a
// dense run takes 165 against 237 us, of uniform keys 54 against 54, of five keys
// over and over 63 against 56 (the other sort is fastest there: 12 us against 21).
constexpr u32 kSmallMax = 12288;

constexpr u32 kRankKeys = 32;     // keys ranked by a workgroup of 256
constexpr u32 kSliceKeys = 255;   // keys of a slice unit (and the one before them)
static_assert((kSmallMax + kSliceKeys - 1) / kSliceKeys <= kSmallParts, "one part per unit");

template <typename K>
struct RankSmem {
  static constexpr u32 C = 16384 / sizeof(K);   // batch keys compared per round
  K k[C];
};

// Keys [32 unit, 32 unit + 32) to their places in the stable order of the n
// keys, with their values (vals may be null).  A wave holds eight keys in
// scalar registers and its lanes share the comparisons, so each batch key read
// from LDS serves eight (eight lanes per key, a read per comparison, left LDS
// the bound: 42 us for 16384 u64 keys, 31 so).  All 256 threads call.
template <typename K>
__device__ __forceinline__ void rank_unit(const K* __restrict__ keys, const K* __restrict__ vals,
                                          u32 n, u32 unit, K* __restrict__ ok, K* __restrict__ ov,
                                          RankSmem<K>& sm) {
  constexpr u32 C = RankSmem<K>::C, E = 16 / sizeof(K), Q = kRankKeys / 4;
  constexpr u32 G = 64 * E;   // keys a wave compares per step
  const u32 tid = threadIdx.x, lane = tid & 63u;
  const u32 i0 = unit * kRankKeys;
  const u32 iw = i0 + Q * (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  K x[Q];
  u32 rank[Q];
#pragma unroll
  for (u32 q = 0; q < Q; ++q) {
    x[q] = iw + q < n ? keys[iw + q] : K(0);
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
      if (c0 + r * 256 < n) buf[r] = j < n ? keys[j] : key_max<K>();
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
    const u32 at = lane * E;
#pragma unroll 2
    for (u32 j = at; j < lo; j += G) {
      const KeyVec<K, (int)E> v = *reinterpret_cast<const KeyVec<K, (int)E>*>(&sm.k[j]);
#pragma unroll
      for (u32 q = 0; q < Q; ++q)
#pragma unroll
        for (u32 e = 0; e < E; ++e) rank[q] += v.k[e] <= x[q] ? 1u : 0u;
    }
    for (u32 j = lo + at; j < mid; j += G) {
      const KeyVec<K, (int)E> v = *reinterpret_cast<const KeyVec<K, (int)E>*>(&sm.k[j]);
#pragma unroll
      for (u32 q = 0; q < Q; ++q)
#pragma unroll
        for (u32 e = 0; e < E; ++e)
          rank[q] += (v.k[e] < x[q] || (v.k[e] == x[q] && c0 + j + e < iw + q)) ? 1u : 0u;
    }
#pragma unroll 2
    for (u32 j = mid + at; j < cpad; j += G) {
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
  if (lane < Q && iw + lane < n && mine < n) {
    ok[mine] = xm;
    if (vals) ov[mine] = vals[iw + lane];
  }
}

// Sort of one list (grid: its units).  Block 0 clears the counter of the
// workgroup-wide items of the update call this starts (ctl may be null).
template <typename K>
__global__ __launch_bounds__(256) void k_rank_sort(const K* __restrict__ keys,
                                                   const K* __restrict__ vals, u32 n,
                                                   K* __restrict__ ok, K* __restrict__ ov,
                                                   Ctl* ctl) {
  __shared__ RankSmem<K> sm;
  if (ctl && blockIdx.x == 0 && threadIdx.x == 0) ctl->wide_n = 0;
  rank_unit<K>(keys, vals, n, blockIdx.x, ok, ov, sm);
}

struct SliceUnitSmem {
  u32 b[256];
  u32 live[257];          // live keys before each thread's
  u32 tmp[256 / 64 + 1];
  u64 start[4];           // per wave: keys that begin a slice (or lie past the batch)
  u32 cross_from, cross_to, cross_live;
  u32 bad;
  unsigned long long need;
};

// Work items of keys [255 unit, 255 unit + 255) of a sorted update list:
// a.work[i] is the slice that begins at key i, empty when none does.  INSERT:
// the unit's part of the node bound, exactly the sum of slices_share with
// every slice's live keys counted, goes to ctl->part[unit].  All 256 threads
// call.
template <typename K, bool INSERT>
__device__ __forceinline__ void slice_unit(const SliceArgs<K>& a, const DirTree<K>& t,
                                           const K* s_top, u32 unit, SliceUnitSmem& sm) {
  const u32 tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
  const u32 i = unit * kSliceKeys + tid - 1;      // thread 0: the key before the unit's
  const bool valid = unit * kSliceKeys + tid >= 1 && i < a.m;
  const K x[1] = {valid ? a.skeys[i] : K(0)};
  u32 bb[1];
  find_buckets<K, 1>(t, s_top, a.nb, x, bb);
  const u32 b = valid ? bb[0] : kNil;
  bool live = false;
  if (INSERT && valid && tid > 0) {
    live = i + 1 == a.m || a.skeys[i + 1] != x[0];
    if (a.svals[i] == key_max<K>()) sm.bad = 1;   // (cleared by the caller)
  }
  sm.b[tid] = b;
  if (tid == 0) {
    sm.need = 0;
    sm.cross_from = 0;
    sm.cross_to = 0;
    sm.cross_live = 0;
  }
  __syncthreads();
  const bool start = tid > 0 && (!valid || sm.b[tid - 1] != b);
  const u64 sb = wave_ballot(start);
  if (lane == 0) sm.start[wv] = sb;
  u32 pre = 0, tot = 0;
  if (INSERT) {
    pre = block_exclusive_scan<256>(live ? 1u : 0u, sm.tmp, &tot);
    sm.live[tid] = pre;
    if (tid == 0) sm.live[256] = tot;
  }
  __syncthreads();
  const bool head = start && valid;
  // the next start after this thread, 256 when the unit holds none
  u32 nx = 256;
  {
    u64 m = lane == 63 ? 0ull : sm.start[wv] & (~0ull << (lane + 1));
    u32 w = wv;
    while (!m && ++w < 4) m = sm.start[w];
    if (m) nx = w * 64 + ctz64(m);
  }
  u32 e = 0;
  if (head) {
    e = i + (nx - tid);
    if (nx == 256) {   // the unit's last slice runs on past it
      e = upper_bound_idx<K>(a.skeys, e, a.m, a.mkba[b]);
      if (INSERT) {
        sm.cross_from = i + (256 - tid);
        sm.cross_to = e;
      }
    }
  }
  if (INSERT) {
    __syncthreads();
    const u32 to = sm.cross_to;
    u32 c = 0;
    for (u32 q = sm.cross_from + tid; q < to; q += 256)
      c += (q + 1 == a.m || a.skeys[q + 1] != a.skeys[q]) ? 1u : 0u;
    if (c) atomicAdd(&sm.cross_live, c);
    __syncthreads();
  }
  if (tid > 0 && valid) {
    WorkItem it;
    it.b = b;
    it.s = i;
    it.e = head ? e : i;
    it.head = 0;
    if (head) {
      const u32 len = e - i;
      if (INSERT) {
        const u64 w = *reinterpret_cast<const u64*>(&a.hdr[b].size);
        const u32 size = (u32)w;
        const u32 t_live = sm.live[nx] - pre + (nx == 256 ? sm.cross_live : 0u);
        const u32 f = a.cap / 2;
        unsigned long long need = 0;
        if ((u32)(w >> 32) == kNil) {
          const u64 c = (u64)size + t_live;
          if (c > a.cap) need = c / f - 1;
        } else {
          const u32 bn = a.bnodes[b];
          need = (u64)(bn < t_live ? bn : t_live) + t_live / f;
        }
        if (need) atomicAdd(&sm.need, need);
      }
      // long slices and chains go to the workgroup-wide kernels
      if (a.wide_min &&
          (INSERT ? len >= a.wide_min
                  : len >= kWideDelKeys && wide_delete_item(len, a.bnodes[b], a.wide_min))) {
        const u32 k = atomicAdd(&a.ctl->wide_n, 1u);
        if (k < a.wide_cap) a.wide[k] = it;
        else atomicCAS(&a.ctl->status, 0u, kErrInternal);   // bound violated: never expected
        it.e = i;
      }
    }
    a.work[i] = it;
  }
  if (unit == 0 && tid == 0 && a.snapshot) {
    a.ctl->free_snapshot = a.ctl->free_top;
    a.ctl->need = 0;
    a.ctl->call_err = 0;
    a.ctl->call_abort = 0;
  }
  __syncthreads();
  if (INSERT && tid == 0 && a.parts)
    a.parts[unit] = (u64)sm.need | (sm.bad ? kPartBad : 0ull);
  __syncthreads();
}

template <typename K, bool INSERT>
__global__ __launch_bounds__(256) void k_small_slices(SliceArgs<K> a, DirTree<K> t) {
  __shared__ __align__(16) K s_top[DirTop<K>::n];
  __shared__ SliceUnitSmem sm;
  if (threadIdx.x == 0) sm.bad = 0;
  load_top<K, 256>(t, s_top);
  slice_unit<K, INSERT>(a, t, s_top, blockIdx.x, sm);
}

}  // namespace flix
