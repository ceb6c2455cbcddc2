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
// 2^26 keys 82 us, at nearly 4 L2 misses of 64 bytes per query (header, one or
// two of the node's blocks, value, part of maxBucket: 50 G random 64-byte
// requests/s).  The first block looked at is the one where the query lies
// between the ends of its bucket (bisecting by the last keys of the blocks read
// one more: lookups of 2^20 95 us, 108 on 2^25 u64 keys, now 83, and with 256
// slots per node, now 74).  Against the sorted form before: lookups of 2^20 keys
// 109 -> 82 us, Zipf 300 to 350 -> 60, 256 lookups 22 -> 8 (one launch), 2^20 ranges
// of 16 keys each 918 -> 218 us, 2^16 of 256 keys 236 -> 107.
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
// its own; `valid` may be 0.  quad_fetch issues every load, quad_count counts.
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
template <typename K, int N>
struct QuadBlock {
  KeyVec<K, 16 / (int)sizeof(K)> v[N * sizeof(K) / 16];
};
template <typename K, int N>
__device__ __forceinline__ void quad_fetch(const K* p, u32 lim, QuadBlock<K, N>& r) {
  quad_load<K, N, 0>(p, lim, r.v);
  quad_load<K, N, 1>(p, lim, r.v);
  quad_load<K, N, 2>(p, lim, r.v);
  quad_load<K, N, 3>(p, lim, r.v);
}
template <typename K, int N, bool LE, bool FULL>
__device__ __forceinline__ void quad_count(const QuadBlock<K, N>& r, u32 valid, K x, K y, u32* n_lt,
                                           u32* n_le) {
  u32 lt = 0, le = 0;
  quad_tally<K, N, LE, FULL, 0>(r.v, valid, x, y, lt, le);
  quad_tally<K, N, LE, FULL, 1>(r.v, valid, x, y, lt, le);
  quad_tally<K, N, LE, FULL, 2>(r.v, valid, x, y, lt, le);
  quad_tally<K, N, LE, FULL, 3>(r.v, valid, x, y, lt, le);
  const u32 s = 8u * (threadIdx.x & 3u);
  *n_lt = (quad_sum(lt) >> s) & 0xFFu;
  if (LE) *n_le = (quad_sum(le) >> s) & 0xFFu;
}

// Buckets of Q queries per lane: the first maxBucket entry >= x.  The searches
// of a lane advance together, so Q of its loads are in flight at a time.  All
// lanes of the wave call.  (s_top holds the top level; every level ends in
// KEY_MAX, so an entry >= x exists.)
template <typename K, int Q>
__device__ __forceinline__ void find_buckets(const DirTree<K>& t, const K* s_top, u32 nb,
                                             const K (&x)[Q], u32 (&i)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) i[q] = 0;
  for (u32 s = DirTop<K>::n / 2; s > 0; s >>= 1) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (i[q] + s <= t.ntop && s_top[i[q] + s - 1] < x[q]) i[q] += s;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) i[q] = i[q] < t.ntop ? i[q] : t.ntop - 1;
#pragma unroll
  for (int l = kDirMaxLev - 1; l >= 0; --l) {
    if ((u32)l < t.nlev) {
      QuadBlock<K, (int)kDirFan> e[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q)
        quad_fetch<K, (int)kDirFan>(t.lev[l] + (u64)i[q] * kDirFan, kDirFan, e[q]);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        u32 c, none;
        quad_count<K, (int)kDirFan, false, true>(e[q], kDirFan, x[q], x[q], &c, &none);
        i[q] = i[q] * kDirFan + (c < kDirFan - 1 ? c : kDirFan - 1);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) i[q] = i[q] < nb ? i[q] : nb - 1;
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

__device__ __forceinline__ u32 wave_read(u32 v, int l) {
  return (u32)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ u64 wave_read(u64 v, int l) {
  return ((u64)(u32)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) |
         (u32)__builtin_amdgcn_readlane((int)(u32)v, l);
}

// Queries per wave (q or fewer) of a batch of m ranges on `waves` resident waves.
// A range's results are copied by its wave (16 ranges of 2^18 results in one wave
// took four times as long as in a wave each); but idle lanes cost, too, so a wave
// takes fewer only while the batch then needs at most an eighth of the waves (ten
// calls on 8192 waves, u32: 4096 ranges of up to 16 keys 103 us with four or two per
// wave, 112 with one; 1000 of up to 64 keys 109 with four, 102 with one).
__host__ __device__ inline u32 range_queries_per_wave(u32 q, u32 m, u32 waves) {
  while (q > 1 && (u64)(q / 2) * waves >= 8ull * m) q >>= 1;
  return q;
}

// A range that the whole wave finishes (all fields uniform).
template <typename K>
struct WaveRange {
  K hi;
  u32 b, next;   // bucket of the last node counted, and that node's link
  u32 cnt;       // keys counted
  bool walk;     // follow chains, too (else the lane does)
  bool off;      // the lane goes on alone: at a chain, or at a stretch of empty buckets
  bool end, bad;
};

// The next up to 64 nodes of the range, one per lane (c keys of *node, 0 in the
// lanes that are left): heads of the buckets that follow, a lane each, as far as
// they lie within the range, and links of a chain.
template <typename K>
__device__ __forceinline__ u32 wave_gather(const ReadArgs<K>& a, WaveRange<K>& r, u32* node) {
  const u32 lane = threadIdx.x & 63u;
  u32 c = 0, n = 0;   // n lanes are taken
  while (n < 64 && !r.end && !r.off) {
    if (r.next != kNil) {
      r.off = !r.walk;
      if (r.off) break;
      r.bad = r.bad || r.next >= a.pool;
      if (r.bad) break;
      const NodeHdr h = a.hdr[r.next];
      const u32 size = wave_read(h.size, 0);
      r.bad = size > a.cap;
      if (r.bad) break;
      r.end = wave_ballot(h.fence > (u64)r.hi) != 0;   // a fence bounds its node's keys from above
      u32 take = size;
      if (r.end) take = upper_bound_idx<K>(a.nkeys + (u64)r.next * a.cap, 0u, size, r.hi);
      if (lane == n) {
        *node = r.next;
        c = take;
      }
      r.next = wave_read(h.next, 0);
      ++n;
    } else {
      const u32 i = r.b + 1 + (lane - n);
      const bool in = lane >= n && i < a.nb;
      NodeHdr h;
      h.fence = 0;
      h.size = 0;
      h.next = kNil;
      if (in) h = a.hdr[i];
      const u64 beyond = ~0ull << n;   // lanes not taken yet
      const u64 stop = wave_ballot(!(in && h.fence <= (u64)r.hi)) & beyond;
      const u64 chain = wave_ballot(h.next != kNil) & beyond;
      const u32 ns = stop ? (u32)ctz64(stop) : 64u;
      const u32 nc = chain ? (u32)ctz64(chain) : 64u;
      // up to the first chain's head, or to the bucket that the range ends in
      const u32 last = nc < ns ? nc : ns < 63 ? ns : 63u;
      r.end = nc >= ns && ns < 64;
      const bool mine = lane >= n && lane <= last;
      r.bad = wave_ballot(mine && h.size > a.cap) != 0;
      if (r.bad) break;
      if (mine) {
        *node = i;
        c = h.size;
        if (r.end && lane == last && in)
          c = upper_bound_idx<K>(a.nkeys + (u64)i * a.cap, 0u, h.size, r.hi);
      }
      if (nc < ns) r.next = wave_read(h.next, (int)nc);
      r.b += last + 1 - n;
      r.off = !r.end && nc >= ns && !wave_ballot(mine && c != 0);
      n = last + 1;
    }
  }
  r.end = r.end || r.bad;
  return r.bad ? 0u : c;
}

// Answers of queries j[0..Q) of every lane (live: it exists).  All lanes of
// the wave call.
template <typename K, int OP, int Q>
__device__ __forceinline__ void direct_read(const ReadArgs<K>& a, const DirTree<K>& t,
                                            const K* s_top, const u32 (&j)[Q],
                                            const bool (&live)[Q]) {
  constexpr u32 B = 64 / sizeof(K);
  constexpr bool UPPER = OP == kOpPredecessor;   // bound: first key > x, else >= x
  const K NF = key_max<K>();
  const u32 lane = threadIdx.x & 63u;
  const OccLevels occ = occ_levels(a.occ, a.nb);
  K x[Q], hi[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    x[q] = live[q] ? a.skeys[j[q]] : K(0);
    hi[q] = (OP == kOpRange && live[q]) ? a.hi[j[q]] : x[q];
  }
  u32 b[Q];
  find_buckets<K, Q>(t, s_top, a.nb, x, b);

  // headers of the buckets' head nodes, and the key the bucket begins after
  NodeHdr h0[Q];
  K from[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    h0[q] = a.hdr[b[q]];
    from[q] = b[q] ? a.mkba[b[q] - 1] : K(0);
  }
  // 64-byte blocks [lo, hb] of the node that may hold the bound, and the one to
  // look at first: where the query lies between the ends of the bucket
  u32 node[Q], size[Q], next[Q], lo[Q], hb[Q], m[Q];
  bool single[Q], bad[Q], open[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    node[q] = b[q];
    size[q] = h0[q].size;
    next[q] = h0[q].next;
    single[q] = next[q] == kNil;
    if (!single[q] && OP != kOpPredecessor) {
      NodeHdr h;
      h.size = 0;
      h.next = kNil;
      node[q] = locate_node(a.hdr, a.pool, b[q], (u64)x[q], &h);
      size[q] = h.size;
      next[q] = h.next;
    }
    bad[q] = node[q] == kBadLink || size[q] > a.cap;
    if (bad[q]) {
      node[q] = b[q];
      size[q] = 0;
      next[q] = kNil;
    }
    lo[q] = 0;
    hb[q] = size[q] ? (size[q] - 1) / B : 0u;
    const K width = (K)h0[q].fence - from[q];
    const float part = (float)(K)(x[q] - from[q]) * __builtin_amdgcn_rcpf((float)width);
    const u32 g = single[q] ? (u32)(fminf(part, 1.0f) * (float)size[q]) / B : hb[q] / 2;
    m[q] = g < hb[q] ? g : hb[q];
    open[q] = true;
  }
  // The keys of block m below x (lt) and not above x or hi (le).  When the bound
  // is not in it the neighbour follows, then the middle of what is left.  (A
  // bound at the start of a block may be left at the end of the one before.)
  u32 lt[Q], le[Q], valid[Q];
  u64 at[Q];
  for (u32 step = 0;; ++step) {
    bool any = false;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (quad_sum(open[q] ? 1u : 0u) != 0) {   // whole quads
        QuadBlock<K, (int)B> blk;
        u32 c, d;
        at[q] = (u64)node[q] * a.cap + m[q] * B;
        valid[q] = size[q] - m[q] * B < B ? size[q] - m[q] * B : B;
        quad_fetch<K, (int)B>(a.nkeys + at[q], a.cap, blk);
        quad_count<K, (int)B, true, false>(blk, valid[q], x[q], hi[q], &c, &d);
        lt[q] = c;
        le[q] = d;
        if (open[q]) {
          const u32 in = UPPER ? d : c;
          open[q] = false;
          if (OP == kOpLookup && d > c) {
          } else if (in == valid[q] && m[q] < hb[q]) {
            lo[q] = m[q] + 1;
            m[q] = step == 0 ? lo[q] : (lo[q] + hb[q]) / 2;
            open[q] = true;
          } else if (in == 0 && m[q] > lo[q]) {
            hb[q] = m[q] - 1;
            m[q] = step == 0 ? hb[q] : (lo[q] + hb[q]) / 2;
            open[q] = true;
          }
        }
      }
      any = any || open[q];
    }
    if (!wave_ballot(any)) break;
  }

  if constexpr (OP == kOpRange) {
    // the range's keys node by node: [p, ub) of each, copied by the wave.  A range
    // that has passed more buckets than there are ranges left goes on 64 buckets at
    // a time, taken by the whole wave.  Chains are followed side by side, a lane
    // each (one by one, 2^20 ranges of which a fifth ran through chains of 500 nodes
    // took 3.8 ms, so 1.2); the last range left has its own followed 64 links at a
    // time.  Long ranges are bound by the latency of one wave's loads: one of 2^20
    // u32 results 9.5 ms, of 2^20 u64 14.0 (node by node 18.8 and 18.4, link by link
    // with the wave's other ranges 25 and 28).
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      bool more = live[q] && !bad[q] && x[q] <= hi[q];
      const u64 ob = (u64)j[q] * a.maxpq;
      u32 cnt = 0, p = m[q] * B + lt[q];
      u32 ub = m[q] * B + le[q];
      NodeHdr h;
      h.fence = 0;
      h.size = size[q];
      h.next = next[q];
      if (more && le[q] == valid[q] && ub < h.size)   // every key of the block is in the range
        ub = upper_bound_idx<K>(a.nkeys + (u64)node[q] * a.cap, ub, h.size, hi[q]);
      u32 run = 0;   // buckets passed since the last link of a chain
      WaveRange<K> r;
      int rl = -1;   // lane of the range that the wave finishes
      u64 left;
      for (u32 step = 0; (left = wave_ballot(more)) != 0; ++step) {
        u32 c = 0;
        u64 src, dst;
        if (__builtin_expect(rl < 0 && (step & 3u) == 2u, 0)) {   // (looked at now and then)
          r.walk = (left & (left - 1)) == 0;
          const u64 ready =
              r.walk ? left : wave_ballot(more && h.next == kNil && run > (u32)__popcll(left));
          if (ready) {
            rl = (int)ctz64(ready);
            r.hi = wave_read(hi[q], rl);
            r.b = wave_read(b[q], rl);
            r.next = wave_read(h.next, rl);
            r.cnt = wave_read(cnt, rl);
            r.off = false;
            r.end = false;
            r.bad = false;
          }
        }
        if (__builtin_expect(rl >= 0, 0)) {
          u32 nd = 0;
          const u32 got = wave_gather<K>(a, r, &nd);
          const u32 incl = wave_scan(got);
          const u32 at = r.cnt + incl - got;
          const u32 room = at < a.maxpq ? a.maxpq - at : 0u;
          c = got < room ? got : room;
          src = (u64)nd * a.cap;
          dst = wave_read(ob, rl) + at;
          r.cnt += wave_read(incl, 63);
          if (r.end || r.off) {
            if (lane == (u32)rl) {
              cnt = r.cnt;
              b[q] = r.b;
              h.next = r.next;
              bad[q] = r.bad;
              more = !r.end;
            }
            rl = -1;
          }
        } else {
          if (step > 0 && more) {
            run = h.next == kNil ? run + 1 : 0u;
            NodeHdr g;
            const u32 nn = next_nonempty(a.hdr, occ, a.nb, a.pool, &b[q], h, &g);
            if (nn == kNil || nn == kBadLink || g.size > a.cap) {
              bad[q] = nn != kNil;
              more = false;
            } else {
              node[q] = nn;
              h = g;
              p = 0;
              // a fence bounds its node's keys from above
              ub = h.fence <= (u64)hi[q]
                       ? h.size
                       : upper_bound_idx<K>(a.nkeys + (u64)nn * a.cap, 0u, h.size, hi[q]);
            }
          }
          const u32 got = more ? ub - p : 0u;
          const u32 room = cnt < a.maxpq ? a.maxpq - cnt : 0u;
          c = got < room ? got : room;
          src = (u64)node[q] * a.cap + p;
          dst = ob + cnt;
          cnt += got;
          if (more && ub < h.size) more = false;   // a key above hi ends the range
        }
        if (wave_ballot(c != 0)) wave_copy_runs<K>(a, src, dst, c);   // (else only counted)
      }
      if (live[q]) a.counts[j[q]] = bad[q] ? 0u : cnt;
    }
  } else {
    // slot of the answer, ~0 when there is none
    u64 slot[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (OP == kOpLookup) {
        slot[q] = le[q] > lt[q] ? at[q] + lt[q] : ~0ull;
      } else if (OP == kOpSuccessor) {
        slot[q] = at[q] + lt[q];
        if (m[q] * B + lt[q] >= size[q] && !bad[q]) {   // past the node: the next one that holds a key
          NodeHdr h, g;
          h.next = next[q];
          const u32 nn = next_nonempty(a.hdr, occ, a.nb, a.pool, &b[q], h, &g);
          bad[q] = nn == kBadLink;
          slot[q] = nn == kNil ? ~0ull : (u64)nn * a.cap;
        }
      } else {
        slot[q] = at[q] + le[q] - 1;
        // nothing up to x in the block: the key before it, in the chain or in
        // an earlier bucket (a block after a node's first follows a key <= x)
        if (!bad[q] && (le[q] == 0 || !single[q]) && !(m[q] > 0 && single[q]))
          slot[q] = predecessor_slot<K>(a.hdr, a.nkeys, occ, a.pool, a.cap, b[q], x[q], &bad[q]);
      }
      if (bad[q]) slot[q] = ~0ull;
    }
    K rv[Q], rk[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      rv[q] = NF;
      rk[q] = OP == kOpPredecessor ? K(0) : NF;
      if (slot[q] != ~0ull) {
        if (OP != kOpLookup) rk[q] = a.nkeys[slot[q]];
        // a value is read once, from a random line: a non-temporal load leaves
        // the cache to the lines that are read again
        rv[q] = __builtin_nontemporal_load(&a.nvals[slot[q]]);
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (live[q]) {
        if (OP != kOpLookup) a.out_k[j[q]] = rk[q];
        a.out_v[j[q]] = rv[q];
      }
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (live[q] && bad[q]) atomicCAS(a.err, 0u, kErrInternal);
}

// Whether some answers of a batch are stored over keys that another wave has
// still to read: an output overlaps the keys (ranges: lo).  A point read answered
// in place is safe, its lane has read its key by then; nothing else is, so such a
// batch is answered from a copy of its keys (the sorted forms always do that).
template <typename K>
inline bool answers_over_keys(int op, const void* keys, u64 n,
                                                  const void* out_k, const void* out_v,
                                                  const void* counts, u32 maxpq) {
  const u64 k0 = (u64)keys, k1 = k0 + n * sizeof(K);
  const bool range = op == kOpRange;
  auto over = [&](const void* p, u64 bytes) {
    const u64 o = (u64)p;
    return p && (range || o != k0) && o < k1 && k0 < o + bytes;
  };
  const u64 bytes = (range ? n * maxpq : n) * sizeof(K);
  return over(out_v, bytes) || (op != kOpLookup && over(out_k, bytes)) ||
         (range && over(counts, n * sizeof(u32)));
}

// Key lists kept in scratch: both read lists of an epoch until its apply, or the
// one list of a batch whose answers overlap its keys.
template <typename K>
__global__ __launch_bounds__(256) void k_copy_keys(const K* __restrict__ a, u32 na,
                                                    K* __restrict__ ao, const K* __restrict__ b,
                                                    u32 nb, K* __restrict__ bo) {
  for (u32 i = blockIdx.x * 256 + threadIdx.x; i < na + nb; i += gridDim.x * 256) {
    if (i < na) ao[i] = a[i];
    else bo[i - na] = b[i - na];
  }
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

// qpw queries per wave: 64, for ranges range_queries_per_wave.
template <typename K, int NT, int OP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_read_direct(
    ReadArgs<K> a, DirTree<K> t, u32 qpw) {
  __shared__ __align__(16) K s_top[DirTop<K>::n];
  load_top<K, NT>(t, s_top);
  const u32 lane = threadIdx.x & 63u;
  const u32 j[1] = {(blockIdx.x * (NT / 64) + (threadIdx.x >> 6)) * qpw + lane};
  const bool live[1] = {lane < qpw && j[0] < a.m};
  direct_read<K, OP, 1>(a, t, s_top, j, live);
}

}  // namespace flix
