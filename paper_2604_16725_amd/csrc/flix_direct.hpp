// Read batches answered in input order, one lane per query (the batch is not
// sorted): each lane finds its bucket through the maxBucket directory, then
// its slot in the bucket's node, and writes its answer where its query came
// from, so every load of the batch and every store of the answers is
// coalesced.
//
// The flipped form (flix_read2.hpp) pays for sorting the batch, for passing
// over the whole directory and for scattering the answers, whatever the batch
// holds; that is repaid only by many keys per bucket.  Here the directory is
// searched as a tree of fan-out 16 whose upper levels are sampled from
// maxBucket when a layout is built (1/15 of its size); the top level is held
// in LDS.  One launch takes the place of three.
//
// What bounds it: on a store that fits the L2s (2^18 keys) 2^20 lookups take
// 35 us, about half of it the address unit (the lane-by-lane form of the
// 64-byte block reads, 16 accesses per query instead of 7, took 69 us); on
// 2^26 keys 94 us, at 4.5 L2 misses of 64 bytes per query (header, two or
// three of the node's blocks, value, part of maxBucket: 50 G random
// 64-byte requests/s).  Against the sorted form before: lookups of 2^20 keys
// 109 -> 94 us, Zipf 351 -> 64, 256 lookups 22 -> 10 (one launch), 2^20 ranges
// of 16 keys each 918 -> 223 us, 2^16 of 256 keys 236 -> 107.
#pragma once

#include "flix_device.hpp"
#include "flix_read2.hpp"

namespace flix {

constexpr u32 kDirFan = 16;     // directory entries per search step (64 or 128 bytes)
constexpr int kDirMaxLev = 6;   // levels below the top: 2048 * 16^6 > 2^32

// Entries of the level held in LDS, at most: 16 KB, so that eight workgroups
// of 256 lanes share a CU.
template <typename K>
struct DirTop {
  static constexpr u32 n = 16384 / sizeof(K);
};

// Levels of the directory search: lev[0] is maxBucket, entry i of the level
// above is the last of the 16 entries of group i below.  Every level ends in
// KEY_MAX and is padded with it to whole groups.
template <typename K>
struct DirTree {
  const K* top;
  const K* lev[kDirMaxLev];
  u32 ntop;
  u32 nlev;
};

__host__ __device__ inline u64 dir_round(u64 n) { return (n + kDirFan - 1) / kDirFan * kDirFan; }

// Entries of the levels above maxBucket, for nb buckets.
template <typename K>
__host__ __device__ inline u64 dir_entries(u64 nb) {
  u64 t = 0;
  for (u64 n = nb; n > DirTop<K>::n;) {
    n = (n + kDirFan - 1) / kDirFan;
    t += dir_round(n);
  }
  return t;
}

// The levels of nb buckets, stored one after another from `up`.
template <typename K>
__host__ __device__ inline DirTree<K> dir_tree(const K* mkba, const K* up, u32 nb) {
  DirTree<K> t;
  t.top = mkba;
  t.ntop = nb;
  t.nlev = 0;
  for (int l = 0; l < kDirMaxLev; ++l) t.lev[l] = nullptr;
  for (int l = 0; l < kDirMaxLev && t.ntop > DirTop<K>::n; ++l) {
    t.lev[l] = t.top;
    t.nlev = (u32)l + 1u;
    t.ntop = (t.ntop + kDirFan - 1) / kDirFan;
    t.top = up;
    up += dir_round(t.ntop);
  }
  return t;
}

// One level above `lo` (n_lo entries, whose padding is written here too).
template <typename K>
__global__ void k_dir_level(K* __restrict__ lo, u32 n_lo, K* __restrict__ hi, u32 n_hi) {
  const u32 i = blockIdx.x * blockDim.x + threadIdx.x;
  const u32 pad_lo = (u32)dir_round(n_lo), pad_hi = (u32)dir_round(n_hi);
  if (i < pad_lo - n_lo) lo[n_lo + i] = key_max<K>();
  if (i < pad_hi) {
    const u32 e = i * kDirFan + (kDirFan - 1);
    hi[i] = e < n_lo ? lo[e] : key_max<K>();
  }
}

// ---- quads --------------------------------------------------------------
// Four neighbouring lanes read their four 64-byte blocks together, one block
// per step and 16 bytes per lane: the address unit takes one access per block
// instead of four (a lane reading its own block in four 16-byte loads), and
// the counts of the four queries travel packed in one word.
template <int CTRL>
__device__ __forceinline__ u32 quad_dpp(u32 v) {
  return (u32)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int R>
__device__ __forceinline__ u32 quad_bcast(u32 v) {
  return quad_dpp<R * 0x55>(v);
}
template <int R>
__device__ __forceinline__ u64 quad_bcast(u64 v) {
  return ((u64)quad_dpp<R * 0x55>((u32)(v >> 32)) << 32) | quad_dpp<R * 0x55>((u32)v);
}
__device__ __forceinline__ u32 quad_sum(u32 v) {
  v += quad_dpp<0xB1>(v);   // lanes 1 0 3 2
  v += quad_dpp<0x4E>(v);   // lanes 2 3 0 1
  return v;
}

// Of the first `valid` of N sorted keys at p (16-byte aligned, the first `lim`
// of them readable): how many are below x, and with LE how many are not above
// y.  FULL: all N are valid.  All lanes of the wave call, each with a block of
// its own; `valid` may be 0.  Every load is issued before the first count.
template <typename K, int N, int R>
__device__ __forceinline__ void quad_load(const K* p, u32 lim, KeyVec<K, 16 / (int)sizeof(K)>* v) {
  constexpr int E = 16 / (int)sizeof(K);
  constexpr int W = N / E / 4;   // 16-byte words per lane and block
  const K* pr = reinterpret_cast<const K*>(quad_bcast<R>((u64)p));
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const u32 at = ((u32)w * 4u + (threadIdx.x & 3u)) * E;
    v[R * W + w] = *reinterpret_cast<const KeyVec<K, E>*>(pr + (at < lim ? at : 0u));
  }
}
template <typename K, int N, bool LE, bool FULL, int R>
__device__ __forceinline__ void quad_tally(const KeyVec<K, 16 / (int)sizeof(K)>* v, u32 valid, K x,
                                           K y, u32& lt, u32& le) {
  constexpr int E = 16 / (int)sizeof(K);
  constexpr int W = N / E / 4;
  const u32 vr = FULL ? (u32)N : quad_bcast<R>(valid);
  const K xr = quad_bcast<R>(x);
  const K yr = LE ? quad_bcast<R>(y) : K(0);
  u32 a = 0, b = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const u32 at = ((u32)w * 4u + (threadIdx.x & 3u)) * E;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const bool in = FULL || at + i < vr;
      a += (in && v[R * W + w].k[i] < xr) ? 1u : 0u;
      if (LE) b += (in && v[R * W + w].k[i] <= yr) ? 1u : 0u;
    }
  }
  lt |= a << (8 * R);
  if (LE) le |= b << (8 * R);
}
template <typename K, int N, bool LE, bool FULL>
__device__ __forceinline__ void quad_count(const K* p, u32 lim, u32 valid, K x, K y, u32* n_lt,
                                           u32* n_le) {
  KeyVec<K, 16 / (int)sizeof(K)> v[N * sizeof(K) / 16];
  quad_load<K, N, 0>(p, lim, v);
  quad_load<K, N, 1>(p, lim, v);
  quad_load<K, N, 2>(p, lim, v);
  quad_load<K, N, 3>(p, lim, v);
  u32 lt = 0, le = 0;
  quad_tally<K, N, LE, FULL, 0>(v, valid, x, y, lt, le);
  quad_tally<K, N, LE, FULL, 1>(v, valid, x, y, lt, le);
  quad_tally<K, N, LE, FULL, 2>(v, valid, x, y, lt, le);
  quad_tally<K, N, LE, FULL, 3>(v, valid, x, y, lt, le);
  const u32 s = 8u * (threadIdx.x & 3u);
  *n_lt = (quad_sum(lt) >> s) & 0xFFu;
  if (LE) *n_le = (quad_sum(le) >> s) & 0xFFu;
}

// First of the n (<= DirTop) entries in LDS that is >= x; the last entry is
// KEY_MAX, so one exists.
template <typename K>
__device__ __forceinline__ u32 top_search(const K* s_top, u32 n, K x) {
  u32 pos = 0;
  for (u32 s = DirTop<K>::n / 2; s > 0; s >>= 1) {
    if (pos + s <= n && s_top[pos + s - 1] < x) pos += s;
  }
  return pos < n ? pos : n - 1;
}

// Bucket of x: the first maxBucket entry >= x.  All lanes of the wave call.
template <typename K>
__device__ __forceinline__ u32 find_bucket(const DirTree<K>& t, const K* s_top, u32 nb, K x) {
  u32 i = top_search<K>(s_top, t.ntop, x);
#pragma unroll
  for (int l = kDirMaxLev - 1; l >= 0; --l) {
    if ((u32)l < t.nlev) {
      u32 c, none;
      quad_count<K, kDirFan, false, true>(t.lev[l] + (u64)i * kDirFan, kDirFan, kDirFan, x, x,
                                          &c, &none);
      i = i * kDirFan + (c < kDirFan - 1 ? c : kDirFan - 1);
    }
  }
  return i < nb ? i : nb - 1;
}

// First slot of the 64-byte block of a node that holds the first key >= x
// (UPPER: > x), of its last block if there is none.  Each step reads the last
// key of a block; `mid_key` is the key at slot cap/4 - 1 (the middle of a
// bulk-loaded node), loaded by the caller together with the header, used when
// `have_mid`.
template <typename K, bool UPPER>
__device__ __forceinline__ u32 node_block(const K* keys, u32 cap, u32 size, K x, K mid_key,
                                          bool have_mid) {
  constexpr u32 B = 64 / sizeof(K);
  u32 lo = 0, hi = size ? (size - 1) / B : 0u;
  const u32 q = cap / 4;
  if (have_mid && q >= B && size >= q) {
    if (UPPER ? mid_key <= x : mid_key < x) lo = q / B < hi ? q / B : hi;
    else hi = q / B - 1;
  }
  while (lo < hi) {
    const u32 mid = (lo + hi) >> 1;
    const K k = keys[mid * B + (B - 1)];
    if (UPPER ? k <= x : k < x) lo = mid + 1; else hi = mid;
  }
  return lo * B;
}

// Inclusive scan over the wave.
__device__ __forceinline__ u32 wave_scan(u32 v) {
  const u32 lane = threadIdx.x & 63u;
#pragma unroll
  for (u32 o = 1; o < 64; o <<= 1) {
    const u32 y = (u32)__shfl_up((int)v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}
__device__ __forceinline__ u64 shfl64(u64 v, u32 src) {
  const u32 lo = (u32)__shfl((int)(u32)v, (int)src, 64);
  const u32 hi = (u32)__shfl((int)(u32)(v >> 32), (int)src, 64);
  return ((u64)hi << 32) | lo;
}

// Range results: every lane has a run of c pairs from pool slot `src` on to
// copy to output position `dst` on.  The wave copies them together, one pair
// per lane and step whatever the lengths of the runs (a lane finds the run
// its pair belongs to by searching the scanned lengths), so loads and stores
// are coalesced within a run and short runs leave no lane idle.  All lanes of
// the wave call.
template <typename K>
__device__ __forceinline__ void wave_copy_runs(const ReadArgs<K>& a, u64 src, u64 dst, u32 c) {
  constexpr u32 U = 4;   // pairs per lane in flight
  const u32 lane = threadIdx.x & 63u;
  const u32 incl = wave_scan(c);
  const u32 total = (u32)__shfl((int)incl, 63, 64);
  const u64 ds = src - (u64)(incl - c), dd = dst - (u64)(incl - c);
  for (u32 t0 = 0; t0 < total; t0 += 64 * U) {
    u64 s[U], d[U];
    K kk[U], vv[U];
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      if (t0 + u * 64 < total) {   // uniform over the wave
        const u32 t = t0 + u * 64 + lane;
        u32 own = 0;   // first lane whose inclusive count exceeds t
#pragma unroll
        for (u32 o = 32; o > 0; o >>= 1)
          if ((u32)__shfl((int)incl, (int)(own + o - 1), 64) <= t) own += o;
        own = own < 64u ? own : 63u;
        s[u] = shfl64(ds, own) + t;
        d[u] = shfl64(dd, own) + t;
        if (t < total) {
          if (a.out_k) kk[u] = a.nkeys[s[u]];
          if (a.out_v) vv[u] = a.nvals[s[u]];
        }
      }
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      if (t0 + u * 64 + lane < total) {
        if (a.out_k) a.out_k[d[u]] = kk[u];
        if (a.out_v) a.out_v[d[u]] = vv[u];
      }
    }
  }
}

// Answer of query j (live: it exists).  All lanes of the wave call.
template <typename K, int OP>
__device__ __forceinline__ void direct_read(const ReadArgs<K>& a, const DirTree<K>& t,
                                            const K* s_top, u32 j, bool live) {
  constexpr u32 B = 64 / sizeof(K);
  const K NF = key_max<K>();
  const K x = live ? a.skeys[j] : K(0);
  const K hi = (OP == kOpRange && live) ? a.hi[j] : K(0);
  u32 b = find_bucket<K>(t, s_top, a.nb, x);
  // header (size and next) and the middle key of the bucket's head node
  NodeHdr h;
  u32 node = b;
  const u64 w = *reinterpret_cast<const u64*>(&a.hdr[b].size);
  const K mid = a.nkeys[(u64)b * a.cap + (a.cap / 4 - 1)];
  h.fence = 0;
  h.size = (u32)w;
  h.next = (u32)(w >> 32);
  const bool single = h.next == kNil;
  if (!single && OP != kOpPredecessor) node = locate_node(a.hdr, a.pool, b, (u64)x, &h);
  bool bad = node == kBadLink || h.size > a.cap;
  if (bad) {
    node = b;
    h.size = 0;
    h.next = kNil;
  }
  // slot of x in the node: its 64-byte block, then the keys in it
  const u64 nb0 = (u64)node * a.cap;
  const K* keys = a.nkeys + nb0;
  u32 lt, le;
  const u32 base = node_block<K, OP == kOpPredecessor>(keys, a.cap, h.size, x, mid, single);
  const u32 valid = h.size - base < B ? h.size - base : B;
  quad_count<K, (int)B, true, false>(keys + base, a.cap, valid, x, OP == kOpRange ? hi : x, &lt,
                                     &le);
  const OccLevels occ = occ_levels(a.occ, a.nb);
  const u64 at = nb0 + base;
  if (OP == kOpLookup) {
    K rv = NF;
    // a value is read once, from a random line: a non-temporal load leaves
    // the cache to the lines that are read again
    if (le > lt) rv = __builtin_nontemporal_load(&a.nvals[at + lt]);
    if (live) a.out_v[j] = rv;
  } else if (OP == kOpSuccessor) {
    u64 slot = at + lt;
    if (lt >= valid && !bad) {   // past the node: the next node that holds a key
      NodeHdr g;
      const u32 nn = next_nonempty(a.hdr, occ, a.nb, a.pool, &b, h, &g);
      bad = nn == kBadLink;
      slot = nn == kNil ? ~0ull : (u64)nn * a.cap;
    }
    K rk = NF, rv = NF;
    if (!bad && slot != ~0ull) {
      rk = a.nkeys[slot];
      rv = __builtin_nontemporal_load(&a.nvals[slot]);
    }
    if (live) {
      a.out_k[j] = rk;
      a.out_v[j] = rv;
    }
  } else if (OP == kOpPredecessor) {
    u64 slot = at + le - 1;
    // nothing up to x in the block: the key before it, in the chain or in an
    // earlier bucket (a block after a node's first follows a key <= x)
    if (!bad && (le == 0 || !single)) {
      if (base > 0 && single) slot = at - 1;
      else slot = predecessor_slot<K>(a.hdr, a.nkeys, occ, a.pool, a.cap, b, x, &bad);
    }
    K rk = K(0), rv = NF;
    if (!bad && slot != ~0ull) {
      rk = a.nkeys[slot];
      rv = __builtin_nontemporal_load(&a.nvals[slot]);
    }
    if (live) {
      a.out_k[j] = rk;
      a.out_v[j] = rv;
    }
  } else {
    // the range's keys node by node: [p, ub) of each, copied by the wave
    bool more = live && !bad && x <= hi;
    const u64 ob = (u64)j * a.maxpq;
    u32 cnt = 0, p = base + lt;
    u32 ub = base + le;
    if (more && le == valid && ub < h.size)   // every key of the block is in the range
      ub = upper_bound_idx<K>(keys, ub, h.size, hi);
    while (wave_ballot(more)) {
      const u32 got = more ? ub - p : 0u;
      const u32 room = cnt < a.maxpq ? a.maxpq - cnt : 0u;
      wave_copy_runs<K>(a, (u64)node * a.cap + p, ob + cnt, got < room ? got : room);
      cnt += got;
      if (more && ub < h.size) more = false;   // a key above hi ends the range
      if (more) {
        NodeHdr g;
        const u32 nn = next_nonempty(a.hdr, occ, a.nb, a.pool, &b, h, &g);
        if (nn == kNil || nn == kBadLink || g.size > a.cap) {
          bad = nn != kNil;
          more = false;
        } else {
          node = nn;
          h = g;
          p = 0;
          // a fence bounds its node's keys from above
          ub = h.fence <= (u64)hi
                   ? h.size
                   : upper_bound_idx<K>(a.nkeys + (u64)node * a.cap, 0u, h.size, hi);
        }
      }
    }
    if (live) a.counts[j] = bad ? 0u : cnt;
  }
  if (live && bad) atomicCAS(a.err, 0u, kErrInternal);
}

// The top directory level into LDS.
template <typename K, int NT>
__device__ __forceinline__ void load_top(const DirTree<K>& t, K* s_top) {
  constexpr u32 E = 16 / sizeof(K);
  // whole 16-byte words, then what a directory that is the top level itself
  // may leave over
  const u32 nw = t.ntop / E;
  for (u32 i = threadIdx.x; i < nw; i += NT)
    reinterpret_cast<KeyVec<K, (int)E>*>(s_top)[i] =
        reinterpret_cast<const KeyVec<K, (int)E>*>(t.top)[i];
  for (u32 i = nw * E + threadIdx.x; i < t.ntop; i += NT) s_top[i] = t.top[i];
  __syncthreads();
}

// qpw queries per wave (64, or fewer for a range batch too small to fill the
// chip: the copies of its results then spread over more waves).
template <typename K, int NT, int OP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_read_direct(
    ReadArgs<K> a, DirTree<K> t, u32 qpw) {
  __shared__ __align__(16) K s_top[DirTop<K>::n];
  load_top<K, NT>(t, s_top);
  const u32 lane = threadIdx.x & 63u;
  const u32 j = (blockIdx.x * (NT / 64) + (threadIdx.x >> 6)) * qpw + lane;
  direct_read<K, OP>(a, t, s_top, j, lane < qpw && j < a.m);
}

}  // namespace flix
