// Onesweep LSD radix sort of (key, payload) pairs for gfx950.
//
// The paper sorts every operation batch on the GPU before the bucket kernels
// run (Section 3.3; sort cost in Table 1 and Section 6.4).  The method used
// here is Onesweep (Adinets & Merrill, 2022): one read of the keys builds the
// digit histograms of every pass, then each pass is a single kernel in which
// every tile ranks its items, publishes per-digit counts and obtains its
// global offsets by decoupled look-back over the preceding tiles.  The sort is
// stable, which gives "last occurrence wins" for duplicate insert keys.
//
// Layout for wave64: tile = NT threads x IPT items, items arranged wave-
// striped (item k of lane l in wave w sits at w*64*IPT + k*64 + l), so ranking
// item slots k = 0..IPT-1 in order, lanes in order, reproduces input order.
//
// Look-back status words are 64 bits: [63:34] epoch, [33:32] flag, [31:0]
// count.  The epoch changes for every pass launch, so the status array never
// needs clearing between passes or calls.
#pragma once

#include <hip/hip_ext.h>

#include "flix_device.hpp"

namespace flix {

constexpr u64 kFlagAgg = 1;   // tile-local count published
constexpr u64 kFlagPre = 2;   // inclusive prefix published

__device__ __forceinline__ u64 pack_status(u32 epoch, u64 flag, u32 v) {
  return ((u64)epoch << 34) | (flag << 32) | (u64)v;
}

template <typename K, int RB>
struct RadixShape {
  static constexpr int R = 1 << RB;
  static constexpr int P = (int)((sizeof(K) * 8 + RB - 1) / RB);
};

template <typename K, int RB>
__device__ __forceinline__ u32 digit_of(K k, u32 shift) {
  return (u32)(k >> shift) & ((1u << RB) - 1u);
}

// Digit histograms of all passes in one read of the keys.  Block 0 also
// clears `hist_next`, the histogram slot the next sort call will use.
template <typename K, int RB>
struct HistSmem {
  u32 sh[RadixShape<K, RB>::P * RadixShape<K, RB>::R];
};

// Keys per thread and chunk of the histogram: one chunk's loads are all
// issued before its first count, so a chunk costs one memory round trip.
constexpr int kHistIPT = 16;

// Histogram part `part` of `nparts` (grid-stride over chunks of 256 x
// kHistIPT keys; each of a chunk's kHistIPT loads is coalesced across the
// workgroup).
template <typename K, int RB>
__device__ void radix_hist_part(const K* __restrict__ keys, u32 n, u32* __restrict__ hist,
                                u32 part, u32 nparts, HistSmem<K, RB>& sm) {
  constexpr int R = RadixShape<K, RB>::R;
  constexpr int P = RadixShape<K, RB>::P;
  constexpr u32 CH = 256u * kHistIPT;
  u32* sh = sm.sh;
  for (int i = threadIdx.x; i < P * R; i += 256) sh[i] = 0;
  __syncthreads();
  for (u64 base = (u64)part * CH; base < n; base += (u64)nparts * CH) {
    K kk[kHistIPT];
#pragma unroll
    for (int c = 0; c < kHistIPT; ++c) {
      const u64 i = base + (u64)c * 256u + threadIdx.x;
      kk[c] = i < n ? keys[i] : K(0);
    }
#pragma unroll
    for (int c = 0; c < kHistIPT; ++c) {
      if (base + (u64)c * 256u + threadIdx.x < n) {
#pragma unroll
        for (int p = 0; p < P; ++p) atomicAdd(&sh[p * R + digit_of<K, RB>(kk[c], p * RB)], 1u);
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < P * R; i += 256)
    if (sh[i]) atomicAdd(&hist[i], sh[i]);
  __syncthreads();
}

template <typename K, int RB>
__global__ __launch_bounds__(256) void k_radix_hist(const K* __restrict__ keys, u32 n,
                                                    u32* __restrict__ hist,
                                                    u32* __restrict__ hist_next,
                                                    u32* __restrict__ tile_ctr) {
  constexpr int R = RadixShape<K, RB>::R;
  constexpr int P = RadixShape<K, RB>::P;
  __shared__ HistSmem<K, RB> sm;
  if (blockIdx.x == 0 && hist_next != nullptr)
    for (int i = threadIdx.x; i < P * R; i += 256) hist_next[i] = 0;
  (void)tile_ctr;
  radix_hist_part<K, RB>(keys, n, hist, blockIdx.x, gridDim.x, sm);
}

constexpr u32 kSortCluster = 16;   // tiles per look-back cluster
constexpr u32 kLookWindow = 16;    // statuses read per look-back round trip

// Payload modes.
constexpr int kPayNone = 0;    // keys only
constexpr int kPayIndex = 1;   // payload is u32; vin == nullptr means "input index"
constexpr int kPayValue = 2;   // payload read from vin

template <typename K, typename V, int RB, int NT, int IPT, int PAY>
struct OnesweepSmem {
  K k[NT * IPT];
  V v[PAY == kPayNone ? 1 : NT * IPT];
  u32 wc[NT / 64][1 << RB];
  u32 lstart[1 << RB];
  u32 gbase[1 << RB];
  u32 tmp[NT / 64 + 1];
  u32 trivial;
};

template <typename K, typename V>
struct PassArgs {
  const K* kin;
  const V* vin;
  K* kout;
  V* vout;
  u32 n;
  u32 shift;
  const u32* hist_p;
  u64* status;
  u64* status_cl;
  u32 epoch;
  u32* err;
};

// Items of `digit` in the tiles before `tile` (whose own count `tot` is
// published); publishes the tile's inclusive prefix.
template <int R = 256>
__device__ __forceinline__ u32 look_back(u64* status, u64* status_cl, u32 epoch, u32 tile,
                                         u32 digit, u32 tot, u32* err) {
  // Two-level decoupled look-back for this digit.  Tiles form clusters of
  // CL consecutive tiles; the last tile of a cluster also publishes the
  // cluster's aggregate (or inclusive prefix) once it has read its cluster
  // mates.  A tile sums the published counts of its cluster mates (nearest
  // first, LB per round trip) and then those of earlier clusters, stopping
  // at the first inclusive prefix, so the chain of dependent round trips
  // stays short however many tiles the pass has.
  u32 excl = 0;
  if (tile > 0) {
    const u32 c = tile / kSortCluster;
    const u32 cbeg = c * kSortCluster;
    const bool last_of_cluster = (tile == cbeg + kSortCluster - 1);
    bool done = false;
    bool gave_up = false;
    u32 polls = 0;
    // (1) cluster mates [cbeg, tile)
    u32 pt = tile;
    while (!done && pt > cbeg) {
      u64 win[kLookWindow];
#pragma unroll
      for (u32 w = 0; w < kLookWindow; ++w)
        win[w] = (w < pt - cbeg) ? ld_agent(&status[(u64)(pt - 1 - w) * R + digit]) : 0ull;
      u32 used = 0;
#pragma unroll
      for (u32 w = 0; w < kLookWindow; ++w) {
        if (done || w != used || w >= pt - cbeg) continue;
        u64 s = win[w];
        u32 fl = (u32)(s >> 32) & 3u;
        if ((u32)(s >> 34) != epoch || fl == 0) continue;   // not published yet
        excl += (u32)s;
        ++used;
        if (fl == kFlagPre) done = true;
      }
      pt -= used;
      if (!done && used == 0) {
        // Bounded wait: a predecessor that never publishes is a bug, and the
        // kernel must still end; the error word reports it.
        if (++polls > (1u << 22)) { atomicOr(err, 1u); gave_up = true; break; }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (last_of_cluster && !gave_up)
      st_agent(&status_cl[(u64)c * R + digit],
               pack_status(epoch, done ? kFlagPre : kFlagAgg, excl + tot));
    // (2) earlier clusters [0, c)
    u32 pc = c;
    while (!done && !gave_up && pc > 0) {
      u64 win[kLookWindow];
#pragma unroll
      for (u32 w = 0; w < kLookWindow; ++w)
        win[w] = (w < pc) ? ld_agent(&status_cl[(u64)(pc - 1 - w) * R + digit]) : 0ull;
      u32 used = 0;
#pragma unroll
      for (u32 w = 0; w < kLookWindow; ++w) {
        if (done || w != used || w >= pc) continue;
        u64 s = win[w];
        u32 fl = (u32)(s >> 32) & 3u;
        if ((u32)(s >> 34) != epoch || fl == 0) continue;
        excl += (u32)s;
        ++used;
        if (fl == kFlagPre) done = true;
      }
      pc -= used;
      if (!done && used == 0) {
        if (++polls > (1u << 22)) { atomicOr(err, 1u); gave_up = true; break; }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    st_agent(&status[(u64)tile * R + digit], pack_status(epoch, kFlagPre, excl + tot));
    if (last_of_cluster && !gave_up)
      st_agent(&status_cl[(u64)c * R + digit], pack_status(epoch, kFlagPre, excl + tot));
  }
  return excl;
}

// One tile of one onesweep pass.  Tiles must be processed so that every tile
// a tile waits on is resident or finished: in a plain launch tile = workgroup
// id (workgroups are dispatched in id order); in a persistent grid every
// workgroup walks its tiles in increasing order.
// AGENT: items are read and written at agent scope (no workgroup's L2 then holds
// them, and the next pass of the same launch needs no cache written back or
// invalidated).
template <typename T, bool AGENT>
__device__ __forceinline__ T sweep_ld(const T* p) {
  if constexpr (!AGENT) return *p;
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool AGENT, typename T>
__device__ __forceinline__ void sweep_st(T* p, T v) {
  if constexpr (!AGENT)
    *p = v;
  else
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename K, typename V, int RB, int NT, int IPT, int PAY, bool AGENT = false>
__device__ void onesweep_tile(const PassArgs<K, V>& pa, u32 tile,
                              OnesweepSmem<K, V, RB, NT, IPT, PAY>& sm) {
  constexpr int R = 1 << RB;
  constexpr int WAVES = NT / 64;
  constexpr int TILE = NT * IPT;
  static_assert(R <= NT, "one look-back thread per digit");
  const K* __restrict__ kin = pa.kin;
  const V* __restrict__ vin = pa.vin;
  K* __restrict__ kout = pa.kout;
  V* __restrict__ vout = pa.vout;
  const u32 n = pa.n, shift = pa.shift, epoch = pa.epoch;
  const u32* __restrict__ hist_p = pa.hist_p;
  u64* status = pa.status;
  u64* status_cl = pa.status_cl;
  u32* err = pa.err;
  K* s_k = sm.k;
  V* s_v = sm.v;
  auto& s_wc = sm.wc;
  u32* s_lstart = sm.lstart;
  u32* s_gbase = sm.gbase;
  u32* s_tmp = sm.tmp;
  u32& s_trivial = sm.trivial;

  const u32 tid = threadIdx.x;
  const u32 lane = tid & 63;
  const u32 w = tid >> 6;

  if (tid == 0) s_trivial = 0;
  for (int i = tid; i < WAVES * R; i += NT) (&s_wc[0][0])[i] = 0;
  __syncthreads();
  const u32 tile0 = tile * (u32)TILE;

  // Load items (wave-striped) and this pass's digit counts in one round.
  K key[IPT];
  V pay[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
    if (idx < n) {
      key[k] = sweep_ld<K, AGENT>(&kin[idx]);
      if (PAY == kPayIndex) pay[k] = vin ? sweep_ld<V, AGENT>(&vin[idx]) : (V)idx;
      if (PAY == kPayValue) pay[k] = sweep_ld<V, AGENT>(&vin[idx]);
    } else {
      key[k] = K(0);
      if (PAY != kPayNone) pay[k] = V(0);
    }
  }
  u32 hcount = (tid < (u32)R) ? sweep_ld<u32, AGENT>(&hist_p[tid]) : 0u;

  // Global exclusive digit offsets of this pass, and the trivial-pass test
  // (all keys share one digit: the stable permutation is the identity).
  if (tid < (u32)R && hcount == n) s_trivial = 1;
  u32 htotal;
  u32 hexcl = block_exclusive_scan<NT>(hcount, s_tmp, &htotal);

  if (s_trivial) {  // uniform across the grid: no look-back is needed
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
      if (idx < n) {
        sweep_st<AGENT>(&kout[idx], key[k]);
        if (PAY != kPayNone) sweep_st<AGENT>(&vout[idx], pay[k]);
      }
    }
    __syncthreads();
    return;
  }

  // Stable rank of every item among the same-digit items of its wave.
  u32 rank[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
    bool valid = idx < n;
    u32 d = digit_of<K, RB>(key[k], shift);
    const u64 m = match_digit<RB>(d, wave_ballot(valid));
    u32 below = rank_below(m);
    u32 cnt = __popcll(m);
    u32 base = valid ? s_wc[w][d] : 0u;
    rank[k] = base + below;
    if (valid && below == cnt - 1) s_wc[w][d] = base + cnt;
  }
  __syncthreads();

  // Per-digit totals of the tile; turn the per-wave counts into exclusive
  // prefixes across waves.
  u32 tot = 0;
  if (tid < (u32)R) {
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) {
      u32 c = s_wc[ww][tid];
      s_wc[ww][tid] = tot;
      tot += c;
    }
    // Publish the tile aggregate (tile 0 publishes its inclusive prefix).
    st_agent(&status[(u64)tile * R + tid],
             pack_status(epoch, tile == 0 ? kFlagPre : kFlagAgg, tot));
  }
  u32 dummy;
  u32 lstart = block_exclusive_scan<NT>(tid < (u32)R ? tot : 0u, s_tmp, &dummy);
  if (tid < (u32)R) {
    s_lstart[tid] = lstart;
    s_gbase[tid] = hexcl + look_back<R>(status, status_cl, epoch, tile, tid, tot, err);
  }
  __syncthreads();

  // Local counting sort of the tile into LDS.
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
    if (idx < n) {
      u32 d = digit_of<K, RB>(key[k], shift);
      u32 pos = s_lstart[d] + s_wc[w][d] + rank[k];
      s_k[pos] = key[k];
      if (PAY != kPayNone) s_v[pos] = pay[k];
    }
  }
  __syncthreads();

  // Write out in digit order: consecutive threads write consecutive slots of
  // one digit's run.
  u32 valid_n = (n - tile0) < (u32)TILE ? (n - tile0) : (u32)TILE;
#pragma unroll
  for (u32 r = 0; r < (u32)IPT; ++r) {
    const u32 i = tid + r * (u32)NT;
    if (i < valid_n) {
      K kk = s_k[i];
      u32 d = digit_of<K, RB>(kk, shift);
      u32 g = s_gbase[d] + (i - s_lstart[d]);
      if (g < n) {   // always true for a consistent histogram
        sweep_st<AGENT>(&kout[g], kk);
        if (PAY != kPayNone) sweep_st<AGENT>(&vout[g], s_v[i]);
      }
    }
  }
  __syncthreads();
}

template <typename K, typename V, int RB, int NT, int IPT, int PAY>
__global__ __launch_bounds__(NT) void k_onesweep(PassArgs<K, V> pa) {
  __shared__ OnesweepSmem<K, V, RB, NT, IPT, PAY> sm;
  onesweep_tile<K, V, RB, NT, IPT, PAY>(pa, blockIdx.x, sm);
}

// One pass of a long sort (8-bit digits): the same pass over tiles of 6144 to
// 10240 items.  A tile writes a run of 24 to 40 items per digit on average
// instead of 8: with 2048-item tiles a pass over 2^26 u32 pairs took 945 us
// (1.1 TB/s: 32-byte runs), these take 400 (2.7 TB/s; a copy of the same bytes
// 224).  Keys and payloads go through the same LDS buffer one after the other,
// so two (64-bit) or three (32-bit) workgroups share a CU.  Items per thread
// as measured, pairs of 2^26 u32 / 2^24 u64: 12 492 / 178 us, 16 437 / 200, 20
// 400 / 206 (u64 keys with indexes: 145, 133, 160); 256 and 1024 threads were
// slower at every tile size.
constexpr int kBigNT = 512;
template <typename K, int PAY>
struct BigTile {
  static constexpr int IPT = sizeof(K) == 4 ? 20 : PAY == kPayValue ? 12 : 16;
  static constexpr int N = kBigNT * IPT;
};

template <typename K, typename V, int PAY>
struct BigPassSmem {
  union {
    K k[BigTile<K, PAY>::N];
    V v[PAY == kPayNone ? 1 : BigTile<K, PAY>::N];
  };
  u32 wc[kBigNT / 64][256];
  u32 lstart[256];
  u32 gofs[256];
  u32 tmp[kBigNT / 64 + 1];
  u32 trivial;
};

template <typename K, typename V, int PAY>
__global__ __launch_bounds__(kBigNT) void k_onesweep_big(PassArgs<K, V> pa) {
  constexpr int NT = kBigNT, IPT = BigTile<K, PAY>::IPT, WAVES = NT / 64, R = 256;
  constexpr u32 TILE = BigTile<K, PAY>::N;
  extern __shared__ __align__(16) unsigned char s_raw[];
  BigPassSmem<K, V, PAY>& sm = *reinterpret_cast<BigPassSmem<K, V, PAY>*>(s_raw);
  const u32 tile = blockIdx.x;
  const u32 tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const u32 n = pa.n;
  const u32 tile0 = tile * TILE;
  const u32 nv = n - tile0 < TILE ? n - tile0 : TILE;
  if (tid == 0) sm.trivial = 0;
  for (int i = tid; i < WAVES * R; i += NT) (&sm.wc[0][0])[i] = 0;
  const u32 first = w * 64u * IPT + lane;   // wave-striped, as in onesweep_tile
  K key[IPT];
  V pay[PAY == kPayNone ? 1 : IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 i = first + (u32)k * 64u;
    key[k] = i < nv ? pa.kin[tile0 + i] : K(0);
  }
  if (PAY != kPayNone) {
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const u32 i = first + (u32)k * 64u;
      if (PAY == kPayIndex && pa.vin == nullptr) pay[k] = (V)(tile0 + i);
      else pay[k] = i < nv ? pa.vin[tile0 + i] : V(0);
    }
  }
  const u32 hcount = tid < (u32)R ? pa.hist_p[tid] : 0u;
  __syncthreads();
  if (tid < (u32)R && hcount == n) sm.trivial = 1;
  u32 htotal;
  const u32 hexcl = block_exclusive_scan<NT>(hcount, sm.tmp, &htotal);
  if (sm.trivial) {   // one digit: the stable permutation is the identity
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const u32 i = first + (u32)k * 64u;
      if (i < nv) {
        pa.kout[tile0 + i] = key[k];
        if (PAY != kPayNone) pa.vout[tile0 + i] = pay[k];
      }
    }
    return;
  }
  u32 pos[IPT];   // rank among the wave's items of the digit, then the LDS slot
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const bool valid = first + (u32)k * 64u < nv;
    const u32 d = digit_of<K, 8>(key[k], pa.shift);
    const u64 m = match_digit<8>(d, wave_ballot(valid));
    const u32 below = rank_below(m), cnt = (u32)__popcll(m);
    const u32 base = valid ? sm.wc[w][d] : 0u;
    pos[k] = base + below;
    if (valid && below == cnt - 1) sm.wc[w][d] = base + cnt;
  }
  __syncthreads();
  u32 tot = 0;
  if (tid < (u32)R) {
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) {
      const u32 c = sm.wc[ww][tid];
      sm.wc[ww][tid] = tot;
      tot += c;
    }
    st_agent(&pa.status[(u64)tile * R + tid],
             pack_status(pa.epoch, tile == 0 ? kFlagPre : kFlagAgg, tot));
  }
  u32 dummy;
  const u32 lstart = block_exclusive_scan<NT>(tid < (u32)R ? tot : 0u, sm.tmp, &dummy);
  if (tid < (u32)R) sm.lstart[tid] = lstart;
  __syncthreads();
  // the tile's keys in digit order in LDS, while other tiles publish
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if (first + (u32)k * 64u < nv) {
      const u32 d = digit_of<K, 8>(key[k], pa.shift);
      pos[k] += sm.lstart[d] + sm.wc[w][d];
      sm.k[pos[k]] = key[k];
    }
  }
  if (tid < (u32)R)
    sm.gofs[tid] = hexcl + look_back(pa.status, pa.status_cl, pa.epoch, tile, tid, tot, pa.err) -
                   lstart;
  __syncthreads();
  u32 g[IPT];   // output slot of item tid + r * NT of the digit order
#pragma unroll
  for (int r = 0; r < IPT; ++r) {
    const u32 i = tid + (u32)r * NT;
    g[r] = 0xFFFFFFFFu;
    if (i < nv) {
      const K kk = sm.k[i];
      g[r] = sm.gofs[digit_of<K, 8>(kk, pa.shift)] + i;
      if (g[r] < n) pa.kout[g[r]] = kk;   // always true for a consistent histogram
    }
  }
  if (PAY != kPayNone) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < IPT; ++k)
      if (first + (u32)k * 64u < nv) sm.v[pos[k]] = pay[k];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IPT; ++r)
      if (g[r] < n) pa.vout[g[r]] = sm.v[tid + (u32)r * NT];
  }
}

// ---------------------------------------------------------------------------
// Batches of at most kSplitMaxItems items with 8-bit digits: three launches
// and no device-wide look-back chain.
//   k_key_span:   smallest and largest key of the batch, per workgroup;
//   k_tile_split: every tile of kSplitTile items is split stably in LDS into the
//     256ths of that span and written back in place, with the start
//     of every digit inside the tile (one 256-entry row per tile);
//   k_run_sort:   one workgroup per digit.  It reads its column of the row
//     table (where its segment lies in every tile), publishes the run's
//     length, gathers the segments in tile order (a stable concatenation),
//     sorts the run in LDS and writes it at the sum of the lengths published
//     by the lower digits.  A batch with a run longer than LDS holds is sorted
//     by further workgroups of the launch (spill_sort).
// A workgroup only waits on lower workgroups, which were dispatched before it
// and publish before they wait on anything.
constexpr int kLocalNT = 1024;
constexpr int kLocalIPT = 8;
constexpr u32 kLocalCap = kLocalNT * kLocalIPT;

struct LocalSortHead {
  u32 wc[kLocalNT / 64][256];   // per-wave digit counts, then their prefixes
  u32 dstart[256];              // first slot of every digit in the run
  u32 tmp[kLocalNT / 64 + 1];
  u32 range[2];
};
constexpr size_t kLocalHeadBytes = (sizeof(LocalSortHead) + 15) & ~size_t(15);

constexpr int kSplitNT = 512;
constexpr int kSplitIPT = 4;
constexpr u32 kSplitTile = kSplitNT * kSplitIPT;
constexpr u32 kSplitMaxTiles = 1024;
// Runs average n / 256 items and must stay below kLocalCap: 7168 is twelve
// standard deviations of a uniform batch away.
constexpr u32 kSplitMaxItems = 7168 * 256;
static_assert(kSplitMaxItems <= kSplitMaxTiles * kSplitTile, "row table");
constexpr u32 kSpanParts = 256;
static_assert(kSplitMaxTiles <= (u32)kLocalNT, "one tile per thread of a run workgroup");
static_assert(kSplitTile <= 65536u, "segment starts are 16-bit");

// Smallest and largest of the workgroup's keys (lo and hi per thread, KEY_MAX
// and 0 in threads without any), to every thread.  red: 2 * NT / 64 words.  All
// threads call.
template <typename K, int NT>
__device__ __forceinline__ void block_span(K& lo, K& hi, u64* red) {
  constexpr u32 NW = NT / 64;
  const u32 tid = threadIdx.x;
  u64 a = (u64)lo, b = (u64)hi;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const u64 x = __shfl_xor((unsigned long long)a, off, 64);
    const u64 y = __shfl_xor((unsigned long long)b, off, 64);
    a = a < x ? a : x;
    b = b > y ? b : y;
  }
  __syncthreads();
  if ((tid & 63u) == 0) {
    red[tid >> 6] = a;
    red[NW + (tid >> 6)] = b;
  }
  __syncthreads();
  a = red[tid & (NW - 1)];
  b = red[NW + (tid & (NW - 1))];
#pragma unroll
  for (int off = NW / 2; off >= 1; off >>= 1) {
    const u64 x = __shfl_xor((unsigned long long)a, off, 64);
    const u64 y = __shfl_xor((unsigned long long)b, off, 64);
    a = a < x ? a : x;
    b = b > y ? b : y;
  }
  lo = (K)a;
  hi = (K)b;
}

// Counters of spill_sort; k_key_span clears them.
struct SpillCtl {
  u32 hist[8 * 256];
  u32 ticket[16];        // [0]: work handed out
  // finished parts of the reading and of every pass: counted in 16 groups, then
  // the full groups, counters of one line each (a pass over 300000 items 17 us;
  // with one counter for all 23)
  u32 done[9][17][16];
};

// Digits are taken from the span of the batch, not from the key width: keys
// below 2^56, say consecutive numbers, would share their top byte (2^20 such
// u64 keys: one run, sorted by one workgroup in 9 ms; 51 us so).  parts: [256]
// smallest, [256] largest.
template <typename K>
__global__ __launch_bounds__(256) void k_key_span(const K* __restrict__ keys, u32 n,
                                                  u64* __restrict__ parts, SpillCtl* sc, Ctl* ctl) {
  __shared__ u64 red[8];
  if (blockIdx.x == gridDim.x - 1)
    for (u32 i = threadIdx.x; i < sizeof(SpillCtl) / 4; i += 256) reinterpret_cast<u32*>(sc)[i] = 0;
  // the counters of the update call this sort begins (ctl may be null)
  if (ctl && blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      ctl->need = 0;
      ctl->call_err = 0;
      ctl->call_abort = 0;
    }
    reset_work_regions(ctl, threadIdx.x);
  }
  constexpr u32 U = 8;
  K lo = key_max<K>(), hi = K(0);
  for (u64 base = (u64)blockIdx.x * 256 * U; base < n; base += (u64)gridDim.x * 256 * U) {
    K k[U];
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u64 i = base + u * 256 + threadIdx.x;
      k[u] = keys[i < n ? i : base];
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      lo = k[u] < lo ? k[u] : lo;
      hi = k[u] > hi ? k[u] : hi;
    }
  }
  block_span<K, 256>(lo, hi, red);
  if (threadIdx.x == 0) {
    parts[blockIdx.x] = (u64)lo;
    parts[kSpanParts + blockIdx.x] = (u64)hi;
  }
}

// Which 256th of the span [kmin, kmax] a key lies in (of its top 16 bits, scaled,
// so that all 256 are used whatever the span).
template <typename K>
struct SpanDigit {
  K kmin;
  u32 shift, scale;
  __device__ __forceinline__ SpanDigit(K lo, K hi) : kmin(lo) {
    const u64 span = (u64)(K)(hi - lo);
    const u32 width = span ? 64u - (u32)__builtin_clzll(span) : 0u;
    shift = width > 16 ? width - 16 : 0u;
    scale = (1u << 24) / ((u32)(span >> shift) + 1u);
  }
  __device__ __forceinline__ u32 operator()(K k) const {
    return (((u32)((K)(k - kmin) >> shift) & 0xFFFFu) * scale) >> 16;
  }
};

template <typename K, typename V, int PAY>
struct SplitSmem {
  K k[kSplitTile];
  V v[PAY == kPayNone ? 1 : kSplitTile];
  u32 wc[kSplitNT / 64][256];
  u32 lstart[256];
  u32 tmp[kSplitNT / 64 + 1];
  u64 red[2 * kSplitNT / 64];
};

template <typename K, typename V, int PAY>
__global__ __launch_bounds__(kSplitNT) void k_tile_split(const K* __restrict__ kin,
                                                         const V* __restrict__ vin,
                                                         K* __restrict__ ks, V* __restrict__ vs,
                                                         u32* __restrict__ toff, u32 n,
                                                         const u64* __restrict__ parts,
                                                         u32 nparts) {
  __shared__ SplitSmem<K, V, PAY> sm;
  constexpr int IPT = kSplitIPT;
  constexpr int NT = kSplitNT;
  constexpr int WAVES = NT / 64;
  const u32 tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const u32 tile0 = blockIdx.x * kSplitTile;
  for (u32 i = tid; i < (u32)WAVES * 256u; i += NT) (&sm.wc[0][0])[i] = 0;
  K key[IPT];
  V pay[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
    key[k] = K(0);
    if (PAY != kPayNone) pay[k] = V(0);
    if (idx < n) {
      key[k] = kin[idx];
      if (PAY == kPayIndex) pay[k] = vin ? vin[idx] : (V)idx;
      if (PAY == kPayValue) pay[k] = vin[idx];
    }
  }
  // the batch's span, from its parts
  K kmin = key_max<K>(), kmax = K(0);
  if (tid < nparts) {
    kmin = (K)parts[tid];
    kmax = (K)parts[kSpanParts + tid];
  }
  block_span<K, NT>(kmin, kmax, sm.red);
  const SpanDigit<K> dig(kmin, kmax);
  // stable rank among the same-digit items of the wave (wave-striped order)
  u32 rank[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
    const bool valid = idx < n;
    const u32 d = dig(key[k]);
    const u64 m = match_digit<8>(d, wave_ballot(valid));
    const u32 below = rank_below(m);
    const u32 cnt = (u32)__popcll(m);
    const u32 base = valid ? sm.wc[w][d] : 0u;
    rank[k] = base + below;
    if (valid && below == cnt - 1) sm.wc[w][d] = base + cnt;
  }
  __syncthreads();
  u32 tot = 0;
  if (tid < 256u) {
    u32 c[WAVES];
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) c[ww] = sm.wc[ww][tid];
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) {
      sm.wc[ww][tid] = tot;
      tot += c[ww];
    }
  }
  u32 dummy;
  const u32 ls = block_exclusive_scan<NT>(tid < 256u ? tot : 0u, sm.tmp, &dummy);
  if (tid < 256u) {
    sm.lstart[tid] = ls;
    toff[(u64)blockIdx.x * 256u + tid] = ls;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 idx = tile0 + w * 64u * IPT + (u32)k * 64u + lane;
    if (idx < n) {
      const u32 d = dig(key[k]);
      const u32 pos = sm.lstart[d] + sm.wc[w][d] + rank[k];
      sm.k[pos] = key[k];
      if (PAY != kPayNone) sm.v[pos] = pay[k];
    }
  }
  __syncthreads();
  const u32 valid_n = (n - tile0) < kSplitTile ? (n - tile0) : kSplitTile;
#pragma unroll
  for (int r = 0; r < IPT; ++r) {
    const u32 i = tid + (u32)r * NT;
    if (i < valid_n) {
      ks[tile0 + i] = sm.k[i];
      if (PAY != kPayNone) vs[tile0 + i] = sm.v[i];
    }
  }
}

// Where one digit's run lies in the split tiles: segment t starts at
// a[t] inside tile t and holds run positions [p[t], p[t+1]).
struct RunMap {
  u32 p[kSplitMaxTiles + 1];
  unsigned short a[kSplitMaxTiles];
  u64 red[2 * kLocalNT / 64];
};
constexpr size_t kRunMapBytes = (sizeof(RunMap) + 15) & ~size_t(15);

template <typename K, typename V, int PAY>
constexpr size_t run_sort_lds() {
  return kLocalHeadBytes + kRunMapBytes + (size_t)kLocalCap * sizeof(K) +
         (PAY == kPayNone ? 0 : (size_t)kLocalCap * sizeof(V));
}

// Staging index of run position i (0 <= i < run length): the segment is the
// last tile whose first position is <= i (empty segments share positions).
__device__ __forceinline__ u32 run_src(const RunMap& m, u32 ntiles, u32 i) {
  u32 lo = 0, hi = ntiles;   // p[lo] <= i < p[hi]
  while (hi - lo > 1) {
    const u32 mid = (lo + hi) >> 1;
    if (m.p[mid] <= i) lo = mid; else hi = mid;
  }
  return lo * kSplitTile + m.a[lo] + (i - m.p[lo]);
}

// The map of digit d's run; returns its length.  All threads call.
__device__ __forceinline__ u32 load_run_map(const u32* __restrict__ toff, u32 d, u32 n, RunMap& m,
                                            u32* tmp, u32* err) {
  const u32 tid = threadIdx.x;
  const u32 ntiles = (n + kSplitTile - 1) / kSplitTile;   // <= kSplitMaxTiles = blockDim
  u32 c = 0;
  if (tid < ntiles) {
    const u32 tn = (n - tid * kSplitTile) < kSplitTile ? (n - tid * kSplitTile) : kSplitTile;
    const u32 a = toff[(u64)tid * 256u + d];
    const u32 b = d < 255u ? toff[(u64)tid * 256u + d + 1u] : tn;
    if (a <= b && b <= tn) {
      c = b - a;
    } else {   // rows inconsistent with the tiles: never expected
      atomicOr(err, 2u);
    }
    m.a[tid] = (unsigned short)a;
  }
  u32 cnt;
  const u32 pre = block_exclusive_scan<kLocalNT>(c, tmp, &cnt);
  if (tid < ntiles) m.p[tid] = pre;
  if (tid == 0) m.p[ntiles] = cnt;
  return cnt;
}

// Moves item k of every lane (wave-striped, ipt items per lane: position
// w*64*ipt + k*64 + lane) to position to[k]; the items are then held in the
// same layout and lie in s_k / s_v.  All threads call.
template <typename K, typename V, int PAY>
__device__ __forceinline__ void run_exchange(K (&key)[kLocalIPT], V (&pay)[kLocalIPT],
                                             const u32 (&to)[kLocalIPT], u32 cnt, u32 ipt, K* s_k,
                                             V* s_v) {
  const u32 w = threadIdx.x >> 6, lane = threadIdx.x & 63u;
#pragma unroll
  for (int k = 0; k < kLocalIPT; ++k) {
    if ((u32)k < ipt && w * 64u * ipt + (u32)k * 64u + lane < cnt) {
      s_k[to[k]] = key[k];
      if (PAY != kPayNone) s_v[to[k]] = pay[k];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kLocalIPT; ++k) {
    const u32 li = w * 64u * ipt + (u32)k * 64u + lane;
    if ((u32)k < ipt && li < cnt) {
      key[k] = s_k[li];
      if (PAY != kPayNone) pay[k] = s_v[li];
    }
  }
}

// One stable counting pass on the 8-bit digit of (key - kmin) >> shift over
// cnt items held wave-striped.  All threads call.
template <typename K, typename V, int PAY>
__device__ __forceinline__ void run_digit_pass(K (&key)[kLocalIPT], V (&pay)[kLocalIPT], u32 cnt,
                                               u32 ipt, K kmin, u32 shift, LocalSortHead& h,
                                               K* s_k, V* s_v) {
  constexpr int IPT = kLocalIPT;
  constexpr int WAVES = kLocalNT / 64;
  const u32 tid = threadIdx.x, w = tid >> 6, lane = tid & 63u;
  u32 rank[IPT];
  for (u32 i = tid; i < (u32)WAVES * 256u; i += kLocalNT) (&h.wc[0][0])[i] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    rank[k] = 0;
    if ((u32)k < ipt) {   // uniform across the workgroup
      const u32 li = w * 64u * ipt + (u32)k * 64u + lane;
      const bool valid = li < cnt;
      const u32 d = digit_of<K, 8>((K)(key[k] - kmin), shift);
      const u64 vm = wave_ballot(valid);
      if (vm) {
        const u64 m = match_digit<8>(d, vm);
        const u32 below = rank_below(m);
        const u32 c = (u32)__popcll(m);
        const u32 base = valid ? h.wc[w][d] : 0u;
        rank[k] = base + below;
        if (valid && below == c - 1) h.wc[w][d] = base + c;
      }
    }
  }
  __syncthreads();
  u32 tot = 0;
  if (tid < 256u) {
    u32 c[WAVES];
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) c[ww] = h.wc[ww][tid];
#pragma unroll
    for (int ww = 0; ww < WAVES; ++ww) {
      h.wc[ww][tid] = tot;
      tot += c[ww];
    }
  }
  u32 dummy;
  const u32 ds = block_exclusive_scan<kLocalNT>(tid < 256u ? tot : 0u, h.tmp, &dummy);
  if (tid < 256u) h.dstart[tid] = ds;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 li = w * 64u * ipt + (u32)k * 64u + lane;
    if ((u32)k < ipt && li < cnt) {
      const u32 d = digit_of<K, 8>((K)(key[k] - kmin), shift);
      rank[k] += h.dstart[d] + h.wc[w][d];
    }
  }
  run_exchange<K, V, PAY>(key, pay, rank, cnt, ipt, s_k, s_v);
}

// Sorts cnt items held wave-striped whose keys lie in [kmin, kmax].  The top 16
// bits of the span come first, in two passes; few keys of a run agree in them,
// and those are put in order by comparing neighbours in LDS.  Where more than
// kTieMax agree, the whole span is sorted digit by digit.  (Every digit that
// varied, seven of a u64 run: 46 us for the run sort of 2^20 keys, 35 so.)
// Leaves the keys in s_k too.  All threads call.
constexpr u32 kTieMax = 16;

template <typename K, typename V, int PAY>
__device__ __forceinline__ void run_span_sort(K (&key)[kLocalIPT], V (&pay)[kLocalIPT], u32 cnt,
                                              u32 ipt, K kmin, K kmax, LocalSortHead& h, K* s_k,
                                              V* s_v) {
  constexpr int IPT = kLocalIPT;
  const u32 tid = threadIdx.x, w = tid >> 6, lane = tid & 63u;
  const u64 span = (u64)(K)(kmax - kmin);
  const u32 width = span ? 64u - (u32)__builtin_clzll(span) : 1u;
  const u32 sh = width > 16 ? width - 16 : 0u;
  u32 s = sh;
  bool whole = false;   // the digits from the lowest on
  while (true) {
    __syncthreads();
    run_digit_pass<K, V, PAY>(key, pay, cnt, ipt, kmin, s, h, s_k, s_v);
    s += 8;
    if (s < width) continue;
    if (sh == 0 || whole) return;
    // every item looks for its neighbours with the same 16 bits
    if (tid == 0) {
      h.range[0] = 0;
      h.range[1] = 0;
    }
    __syncthreads();
    u32 to[IPT];
    bool tied = false, many = false;
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const u32 li = w * 64u * ipt + (u32)k * 64u + lane;
      to[k] = li;
      if ((u32)k < ipt && li < cnt) {
        const K p = (K)(key[k] - kmin) >> sh;
        u32 before = 0;   // items of the group that belong before this one
        u32 a = li;
        while (a > 0) {
          const K o = s_k[a - 1];
          if (((K)(o - kmin) >> sh) != p) break;
          --a;
          tied = true;
          if (li - a >= kTieMax) { many = true; break; }
          before += o <= key[k] ? 1u : 0u;   // (equal keys keep their order)
        }
        u32 b = li + 1;
        while (b < cnt && !many) {
          const K o = s_k[b];
          if (((K)(o - kmin) >> sh) != p) break;
          ++b;
          tied = true;
          if (b - li > kTieMax) { many = true; break; }
          before += o < key[k] ? 1u : 0u;
        }
        to[k] = a + before;
      }
    }
    if (wave_ballot(tied) && lane == 0) h.range[0] = 1;
    if (wave_ballot(many) && lane == 0) h.range[1] = 1;
    __syncthreads();
    const bool any_tied = h.range[0] != 0, any_many = h.range[1] != 0;
    if (any_many) {
      whole = true;
      s = 0;
      continue;
    }
    if (any_tied) run_exchange<K, V, PAY>(key, pay, to, cnt, ipt, s_k, s_v);
    return;
  }
}

// Length published for digit i (0 if it never is: a bug, and the kernel must
// still end; the error word reports it).
__device__ __forceinline__ u32 wait_run_length(const u64* status, u32 i, u32 epoch, u32* err) {
  u32 polls = 0;
  while (true) {
    const u64 s = ld_agent(&status[i]);
    if ((u32)(s >> 34) == epoch && ((s >> 32) & 3u) != 0u) return (u32)s;
    if (++polls > (1u << 22)) {
      atomicOr(err, 1u);
      return 0;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// A batch with a run longer than kLocalCap items (keys in a few dense stretches,
// or many equal ones) is sorted digit by digit instead, from the split tiles, by
// the further workgroups of the launch: one reading counts every digit, then a
// onesweep pass per digit that varies.  The work is handed out by a counter in
// the order of the passes, so a workgroup waits only on work that a running one
// holds; a pass begins when the one before has ended (its tiles are counted) and
// its data are at agent scope.  Its cost does not depend on the keys: 2^20 u64
// pairs in 64 dense stretches 333 us, 70% one key 320, seven keys 91 (each long
// run by one workgroup: 381, 1133, 4861).  A pass is 36 us there, 17 us of it the
// chain of hand-outs and look-backs, the rest the traffic past the L2: with plain
// stores and a release fence per tile a pass took 48, with fences in every wave 150.
constexpr int kSpillIPT = 4;
constexpr u32 kSpillTile = kLocalNT * kSpillIPT;
constexpr u32 kSpillHistParts = 64;

template <typename K, typename V, int PAY>
using SpillTile = OnesweepSmem<K, V, 8, kLocalNT, kSpillIPT, PAY>;

struct SpillSmem {   // in front of the pass's tile
  u32 hist[8 * 256];
  u32 active[8];   // digits that vary, lowest first
  u32 nactive;
  u32 ticket;
  u32 stop;
};

// Waits until all `parts` are; false when they never are (a bug: the error word
// reports it).  All threads call.
__device__ __forceinline__ bool wait_done(const u32 (*c)[16], u32 parts, SpillSmem& sm, u32* err) {
  if (threadIdx.x == 0) {
    const u32 want = parts < 16u ? parts : 16u;
    u32 polls = 0;
    sm.stop = 0;
    while (ld_agent32(&c[0][0]) < want) {
      if (++polls > (1u << 22)) {
        atomicOr(err, 1u);
        sm.stop = 1;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
  return sm.stop == 0;
}

// Counts part i of `parts` as finished once the workgroup's writes are done.  All
// threads call.
__device__ __forceinline__ void count_done(u32 (*c)[16], u32 i, u32 parts) {
  __builtin_amdgcn_s_waitcnt(0);   // this wave's writes, all at agent scope, are done
  __syncthreads();
  if (threadIdx.x == 0) {
    const u32 g = i & 15u, members = (parts - g + 15u) / 16u;
    if (atomicAdd(&c[1 + g][0], 1u) + 1u == members) atomicAdd(&c[0][0], 1u);
  }
}

// ks / vs: the split tiles, free to overwrite once status[256 + d] of every digit
// is published; xk / xv: as many items; ko / vo: the result.  ps: look-back words
// of the passes, epochs epoch + 1 to epoch + 8.
template <typename K, typename V, int PAY>
__device__ __noinline__ void spill_sort(K* ks, V* vs, K* ko, V* vo, K* xk, V* xv, u64* status,
                                        u64* ps, u64* ps_cl, SpillCtl* sc, u32 epoch, u32 n,
                                        u32* err, unsigned char* lds) {
  constexpr u32 P = (u32)sizeof(K);
  SpillSmem& sm = *reinterpret_cast<SpillSmem*>(lds);
  SpillTile<K, V, PAY>& tm =
      *reinterpret_cast<SpillTile<K, V, PAY>*>(lds + ((sizeof(SpillSmem) + 15) & ~size_t(15)));
  static_assert(sizeof(SpillSmem) + 16 + sizeof(SpillTile<K, V, PAY>) <= run_sort_lds<K, V, PAY>(),
                "the run sort's LDS holds it");
  const u32 tid = threadIdx.x, lane = tid & 63u;
  const u32 tiles = (n + kSpillTile - 1) / kSpillTile;
  const u32 nh = tiles < kSpillHistParts ? tiles : kSpillHistParts;
  bool counted = false, free_ks = false;
  u32 passes = P, next = 0;
  if (tid == 0) next = atomicAdd(&sc->ticket[0], 1u);
  while (true) {
    __syncthreads();
    if (tid == 0) {
      sm.ticket = next;
      next = atomicAdd(&sc->ticket[0], 1u);   // here by the time it is wanted
    }
    __syncthreads();
    const u32 t = sm.ticket;
    if (t < nh) {   // a part of the reading
      for (u32 i = tid; i < P * 256u; i += kLocalNT) sm.hist[i] = 0;
      __syncthreads();
      for (u32 c0 = t * kSpillTile; c0 < n; c0 += nh * kSpillTile) {
        K key[kSpillIPT];
#pragma unroll
        for (int k = 0; k < kSpillIPT; ++k) {
          const u32 i = c0 + (u32)k * kLocalNT + tid;
          key[k] = i < n ? ks[i] : K(0);
        }
#pragma unroll
        for (int k = 0; k < kSpillIPT; ++k) {
          const bool valid = c0 + (u32)k * kLocalNT + tid < n;
          const u64 vm = wave_ballot(valid);
          if (vm == 0) continue;   // uniform over the wave
#pragma unroll
          for (u32 p = 0; p < P; ++p) {
            // a wave's items often share a digit: that of its first lane is
            // counted once
            const u32 d = digit_of<K, 8>(key[k], p * 8);
            const u32 d0 = (u32)__builtin_amdgcn_readfirstlane((int)d);
            const u64 same = wave_ballot(valid && d == d0);
            if (lane == 0) atomicAdd(&sm.hist[p * 256 + d0], (u32)__popcll(same));
            if (valid && d != d0) atomicAdd(&sm.hist[p * 256 + d], 1u);
          }
        }
      }
      __syncthreads();
      for (u32 i = tid; i < P * 256u; i += kLocalNT)
        if (sm.hist[i]) atomicAdd(&sc->hist[i], sm.hist[i]);
      count_done(sc->done[0], t, nh);
      continue;
    }
    if (!counted) {
      if (!wait_done(sc->done[0], nh, sm, err)) return;
      if (tid < P) sm.active[tid] = 1;
      __syncthreads();
      for (u32 i = tid; i < P * 256u; i += kLocalNT)
        if (ld_agent32(&sc->hist[i]) == n) sm.active[i >> 8] = 0;
      __syncthreads();
      if (tid == 0) {
        u32 a = 0;
        for (u32 p = 0; p < P; ++p)
          if (sm.active[p]) sm.active[a++] = p;
        if (a == 0) sm.active[a++] = 0;   // all keys equal: one pass copies them
        sm.nactive = a;
      }
      __syncthreads();
      passes = sm.nactive;
      counted = true;
    }
    const u32 a = (t - nh) / tiles, tile = (t - nh) % tiles;
    if (a >= passes) return;
    if (a > 0 && !wait_done(sc->done[a], tiles, sm, err)) return;
    if (a > 0 && !free_ks) {
      // the run workgroups have read their items out of ks
      if (tid < 256u) (void)wait_run_length(status, 256u + tid, epoch, err);
      free_ks = true;
    }
    const u32 p = sm.active[a];
    const bool last = a + 1 == passes;
    PassArgs<K, V> pa;
    pa.kin = a & 1u ? xk : ks;
    pa.vin = a & 1u ? xv : vs;
    pa.kout = last ? ko : a & 1u ? ks : xk;
    pa.vout = last ? vo : a & 1u ? vs : xv;
    pa.n = n;
    pa.shift = p * 8;
    pa.hist_p = sc->hist + p * 256;
    pa.status = ps;
    pa.status_cl = ps_cl;
    pa.epoch = epoch + 1 + a;
    pa.err = err;
    __syncthreads();
    onesweep_tile<K, V, 8, kLocalNT, kSpillIPT, PAY, true>(pa, tile, tm);
    if (!last) count_done(sc->done[a + 1], tile, tiles);
  }
}

template <typename K, typename V, int PAY>
__global__ __launch_bounds__(kLocalNT) void k_run_sort(K* ks, V* vs, K* ko, V* vo, K* xk, V* xv,
                                                       const u32* __restrict__ toff, u64* status,
                                                       u64* ps_cl, SpillCtl* sc, u32 epoch, u32 n,
                                                       u32* err) {
  extern __shared__ __align__(16) unsigned char lsm[];
  LocalSortHead& h = *reinterpret_cast<LocalSortHead*>(lsm);
  RunMap& m = *reinterpret_cast<RunMap*>(lsm + kLocalHeadBytes);
  K* s_k = reinterpret_cast<K*>(lsm + kLocalHeadBytes + kRunMapBytes);
  V* s_v = reinterpret_cast<V*>(lsm + kLocalHeadBytes + kRunMapBytes +
                                (size_t)kLocalCap * sizeof(K));
  constexpr int IPT = kLocalIPT;
  const u32 tid = threadIdx.x, w = tid >> 6, lane = tid & 63u;
  const u32 ntiles = (n + kSplitTile - 1) / kSplitTile;
  if (blockIdx.x >= 256u) {
    const u32 len = tid < 256u ? wait_run_length(status, tid, epoch, err) : 0u;
    u32 nlong;
    (void)block_exclusive_scan<kLocalNT>(len > kLocalCap ? 1u : 0u, h.tmp, &nlong);
    if (nlong == 0) return;
    __syncthreads();
    spill_sort<K, V, PAY>(ks, vs, ko, vo, xk, xv, status, status + 512, ps_cl, sc, epoch, n, err,
                          lsm);
    return;
  }
  const u32 d = blockIdx.x;
  const u32 cnt = load_run_map(toff, d, n, m, h.tmp, err);
  if (tid == 0) st_agent(&status[d], pack_status(epoch, kFlagAgg, cnt));
  __syncthreads();
  if (cnt == 0 || cnt > kLocalCap) {   // (a long run: the whole batch is sorted above)
    if (tid == 0) st_agent(&status[256u + d], pack_status(epoch, kFlagAgg, 1u));
    return;
  }
  // the run lives in registers and LDS for all of its passes
  K key[IPT], lo = key_max<K>(), hi = K(0);
  V pay[IPT];
  const u32 ipt = (cnt + kLocalNT - 1) / kLocalNT;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 li = w * 64u * ipt + (u32)k * 64u + lane;
    key[k] = K(0);
    if ((u32)k < ipt && li < cnt) {
      const u32 src = run_src(m, ntiles, li);
      key[k] = ks[src];
      if (PAY != kPayNone) pay[k] = vs[src];
    }
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if ((u32)k < ipt && w * 64u * ipt + (u32)k * 64u + lane < cnt) {
      lo = key[k] < lo ? key[k] : lo;
      hi = key[k] > hi ? key[k] : hi;
    }
  }
  block_span<K, kLocalNT>(lo, hi, m.red);
  if (tid == 0) st_agent(&status[256u + d], pack_status(epoch, kFlagAgg, 1u));   // all read
  run_span_sort<K, V, PAY>(key, pay, cnt, ipt, lo, hi, h, s_k, s_v);
  // the sum of the lengths published by the lower digits
  u32 base;
  (void)block_exclusive_scan<kLocalNT>(tid < d ? wait_run_length(status, tid, epoch, err) : 0u,
                                       h.tmp, &base);
  if (base + cnt > n) {   // published lengths inconsistent: never expected
    if (tid == 0) atomicOr(err, 2u);
    return;
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const u32 li = w * 64u * ipt + (u32)k * 64u + lane;
    if ((u32)k < ipt && li < cnt) {
      ko[base + li] = key[k];
      if (PAY != kPayNone) vo[base + li] = pay[k];
    }
  }
}

// Scratch shared by every sort call of one store.
struct SortScratch {
  u32* hist = nullptr;      // [2][P*R] ping-pong histogram slots
  u64* status = nullptr;    // [max_tiles * R]
  u64* status_cl = nullptr; // [max_tiles / cluster * R]
  u32* tile_ctr = nullptr;  // [16] per-pass tile ticket counters (cleared by k_radix_hist)
  u32* err = nullptr;       // sticky sort error bits (1: look-back wait gave up, 2: runs
                            // that do not fit the batch)
  u32 epoch = 0;            // last epoch used
  u32 parity = 0;           // histogram slot of the next call
  u64 max_items = 0;        // capacity of the status array, in items
  u32* toff = nullptr;      // [kSplitMaxTiles][256] digit starts of the split tiles
  u64* span = nullptr;      // [2 * kSpanParts] smallest and largest keys
  SpillCtl* spill = nullptr;
  void* xk = nullptr;       // [x_items] keys between passes of spill_sort (8-byte slots)
  void* xv = nullptr;       // [x_items] their payloads (8-byte slots)
  u64 x_items = 0;
  // optional per-kernel timing hooks (family 0: histogram, 1: one pass or
  // the tile split, 2: the per-run sort):
  // on_begin hands out the start/stop events of the next dispatch
  void (*on_begin)(void* ctx, int family, hipEvent_t* e0, hipEvent_t* e1) = nullptr;
  void (*on_end)(void* ctx, int family, hipEvent_t e0, hipEvent_t e1) = nullptr;
  void* hook_ctx = nullptr;
};

// Kernel launch that, given events, has the dispatch itself stamp them at its
// start and end (hipExtLaunchKernelGGL): timing then adds no marker packets
// between kernels.  Without events it is a plain launch.
template <typename F, typename... Args>
inline void launch_timed(hipEvent_t e0, hipEvent_t e1, F kernel, dim3 grid, dim3 block,
                         uint32_t shm, hipStream_t st, Args... args) {
  if (e0 && e1)
    hipExtLaunchKernelGGL(kernel, grid, block, shm, st, e0, e1, 0u, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, shm, st, args...);
}

struct SortTimer {
  SortScratch& s;
  int fam;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  SortTimer(SortScratch& s_, int fam_) : s(s_), fam(fam_) {
    if (s.on_begin) s.on_begin(s.hook_ctx, fam, &e0, &e1);
  }
  void end() {
    if (s.on_end && e0) s.on_end(s.hook_ctx, fam, e0, e1);
  }
};

// Pass kernel shape: 2048-item tiles of 512 threads x 4 items (eight waves
// share a tile's ranking and scatter; measured faster than 256 x 8 and
// 1024 x 2).  The persistent drain's 256-thread workgroups take the same
// tiles as 256 x 8, so both read the same look-back words.
constexpr int kSortNT = 512;
constexpr int kSortIPT = 4;
constexpr int kSortTile = kSortNT * kSortIPT;
constexpr int kDrainSortNT = 256;
constexpr int kDrainSortIPT = kSortTile / kDrainSortNT;

inline u64 sort_status_words(u64 max_items, int rb) {
  return ((max_items + kSortTile - 1) / kSortTile + 1) * (u64)(1 << rb);
}
inline u64 sort_cluster_words(u64 max_items) {
  return ((max_items + kSortTile - 1) / kSortTile / kSortCluster + 2) * 256ull;
}

// Host driver: sorts n pairs from (kin, vin) using ping-pong buffers
// (k0, v0) / (k1, v1).  Returns which buffer holds the result (0 or 1).
// ctl: control block whose update counters the sort may clear on its way;
// *ctl_reset tells whether it did.
template <typename K, typename V, int RB, int PAY>
hipError_t radix_sort(const K* kin, const V* vin, K* k0, V* v0, K* k1, V* v1, u32 n,
                      SortScratch& s, hipStream_t st, int* result_buf, Ctl* ctl = nullptr,
                      bool* ctl_reset = nullptr) {
  constexpr int R = RadixShape<K, RB>::R;
  constexpr int P = RadixShape<K, RB>::P;
  if (n == 0) {
    *result_buf = 0;
    return hipSuccess;
  }
  if ((u64)n > s.max_items) return hipErrorInvalidValue;
  const u32 ntiles = (n + kSortTile - 1) / kSortTile;
  if (RB == 8 && n <= kSplitMaxItems && s.toff && s.span && s.spill && n <= s.x_items) {
    // three launches: key span, tile split, run sort
    if (s.epoch >= (1u << 30) - 10u) {
      hipError_t e = hipMemsetAsync(s.status, 0, sort_status_words(s.max_items, RB) * sizeof(u64), st);
      if (e != hipSuccess) return e;
      e = hipMemsetAsync(s.status_cl, 0, sort_cluster_words(s.max_items) * sizeof(u64), st);
      if (e != hipSuccess) return e;
      s.epoch = 0;
    }
    const u32 epoch = s.epoch + 1;
    s.epoch += 9;   // the run lengths and up to eight passes
    const u32 nsplit = (n + kSplitTile - 1) / kSplitTile;
    const u32 nparts = (n + 2047) / 2048 < kSpanParts ? (n + 2047) / 2048 : kSpanParts;
    {
      SortTimer t(s, 0);
      launch_timed(t.e0, t.e1, k_key_span<K>, dim3(nparts), dim3(256), 0, st, kin, n, s.span, s.spill,
                   ctl);
      if (ctl_reset) *ctl_reset = ctl != nullptr;
      t.end();
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    {
      SortTimer t(s, 1);
      launch_timed(t.e0, t.e1, k_tile_split<K, V, PAY>, dim3(nsplit), dim3(kSplitNT), 0, st, kin,
                   vin, k0, v0, s.toff, n, (const u64*)s.span, nparts);
      t.end();
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr size_t lds = run_sort_lds<K, V, PAY>();
    static bool lds_set = false;
    if (!lds_set) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_run_sort<K, V, PAY>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      lds_set = true;
    }
    {
      SortTimer t(s, 2);
      // a workgroup per digit and, where a run can be long, as many for
      // spill_sort (one per CU)
      launch_timed(t.e0, t.e1, k_run_sort<K, V, PAY>, dim3(n > kLocalCap ? 512u : 256u),
                   dim3(kLocalNT), (uint32_t)lds, st, k0, v0, k1, v1, (K*)s.xk, (V*)s.xv,
                   (const u32*)s.toff, s.status, s.status_cl, s.spill, epoch, n, s.err);
      t.end();
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    *result_buf = 1;
    return hipSuccess;
  }
  u32* hist = s.hist + (size_t)s.parity * (P * R);
  u32* hist_next = s.hist + (size_t)(s.parity ^ 1u) * (P * R);
  s.parity ^= 1u;
  u32 hb = (n + 256u * kHistIPT - 1u) / (256u * kHistIPT);
  if (hb > 1024u) hb = 1024u;
  {
    SortTimer t(s, 0);
    launch_timed(t.e0, t.e1, k_radix_hist<K, RB>, dim3(hb), dim3(256), 0, st, kin, n, hist,
                 hist_next, s.tile_ctr);
    t.end();
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  for (int p = 0; p < P; ++p) {
    if (s.epoch >= (1u << 30) - 1u) {
      e = hipMemsetAsync(s.status, 0, sort_status_words(s.max_items, RB) * sizeof(u64), st);
      if (e != hipSuccess) return e;
      e = hipMemsetAsync(s.status_cl, 0, sort_cluster_words(s.max_items) * sizeof(u64), st);
      if (e != hipSuccess) return e;
      s.epoch = 0;
    }
    const u32 epoch = ++s.epoch;
    const K* ki = p == 0 ? kin : ((p & 1) ? k0 : k1);
    const V* vi = p == 0 ? vin : ((p & 1) ? v0 : v1);
    K* ko = (p & 1) ? k1 : k0;
    V* vo = (p & 1) ? v1 : v0;
    PassArgs<K, V> pa;
    pa.kin = ki;
    pa.vin = vi;
    pa.kout = ko;
    pa.vout = vo;
    pa.n = n;
    pa.shift = (u32)(p * RB);
    pa.hist_p = hist + p * R;
    pa.status = s.status;
    pa.status_cl = s.status_cl;
    pa.epoch = epoch;
    pa.err = s.err;
    SortTimer t(s, 1);
    if constexpr (RB == 8) {
      constexpr size_t lds = sizeof(BigPassSmem<K, V, PAY>);
      static bool lds_set = false;
      if (!lds_set && lds > 65536) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_onesweep_big<K, V, PAY>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        lds_set = true;
      }
      launch_timed(t.e0, t.e1, k_onesweep_big<K, V, PAY>,
                   dim3((n + BigTile<K, PAY>::N - 1) / BigTile<K, PAY>::N), dim3(kBigNT),
                   (uint32_t)lds, st, pa);
    } else {
      launch_timed(t.e0, t.e1, k_onesweep<K, V, RB, kSortNT, kSortIPT, PAY>, dim3(ntiles),
                   dim3(kSortNT), 0, st, pa);
    }
    t.end();
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  *result_buf = ((P - 1) & 1) ? 1 : 0;
  return hipSuccess;
}

}  // namespace flix
