// Initial build (bulk load), contents dump and the device invariant checker.
#pragma once

#include <algorithm>

#include "flix_device.hpp"
#include "flix_direct.hpp"
#include "flix_occ.hpp"

namespace flix {

// ---------------------------------------------------------------------------
// Stream compaction of a sorted run: keep the LAST item of every equal-key
// run (upsert semantics: the stable sort keeps input order among equal keys).
// Three kernels: per-block counts, one-block scan of the counts, scatter.
// ---------------------------------------------------------------------------
constexpr int kCompactNT = 256;
constexpr int kCompactIPT = 8;
constexpr int kCompactTile = kCompactNT * kCompactIPT;

template <typename K>
__device__ __forceinline__ bool keep_last(const K* k, u64 i, u64 n) {
  return (i + 1 == n) || (k[i] != k[i + 1]);
}

template <typename K>
__global__ __launch_bounds__(kCompactNT) void k_compact_count(const K* __restrict__ k, u64 n,
                                                             u32* __restrict__ bsum) {
  __shared__ u32 s_tmp[kCompactNT / 64 + 1];
  u64 base = (u64)blockIdx.x * kCompactTile + (u64)threadIdx.x * kCompactIPT;
  u32 c = 0;
  for (int j = 0; j < kCompactIPT; ++j) {
    u64 i = base + j;
    if (i < n && keep_last(k, i, n)) ++c;
  }
  u32 tot;
  block_exclusive_scan<kCompactNT>(c, s_tmp, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// One block: exclusive scan of nb block counts in place; total -> *total.
__global__ __launch_bounds__(1024) void k_scan_small(u32* __restrict__ a, u32 nb,
                                                    u32* __restrict__ total) {
  __shared__ u32 s_tmp[1024 / 64 + 1];
  u32 per = (nb + 1023) / 1024;
  u32 beg = threadIdx.x * per;
  u32 sum = 0;
  for (u32 i = beg; i < beg + per && i < nb; ++i) sum += a[i];
  u32 tot;
  u32 ex = block_exclusive_scan<1024>(sum, s_tmp, &tot);
  for (u32 i = beg; i < beg + per && i < nb; ++i) {
    u32 t = a[i];
    a[i] = ex;
    ex += t;
  }
  if (threadIdx.x == 0) *total = tot;
}

template <typename K>
__global__ __launch_bounds__(kCompactNT) void k_compact_scatter(const K* __restrict__ k,
                                                               const K* __restrict__ v, u64 n,
                                                               const u32* __restrict__ boff,
                                                               K* __restrict__ ko,
                                                               K* __restrict__ vo) {
  __shared__ u32 s_tmp[kCompactNT / 64 + 1];
  u64 base = (u64)blockIdx.x * kCompactTile + (u64)threadIdx.x * kCompactIPT;
  u32 c = 0;
  for (int j = 0; j < kCompactIPT; ++j) {
    u64 i = base + j;
    if (i < n && keep_last(k, i, n)) ++c;
  }
  u32 tot;
  u32 pos = block_exclusive_scan<kCompactNT>(c, s_tmp, &tot) + boff[blockIdx.x];
  for (int j = 0; j < kCompactIPT; ++j) {
    u64 i = base + j;
    if (i < n && keep_last(k, i, n)) {
      ko[pos] = k[i];
      vo[pos] = v[i];
      ++pos;
    }
  }
}

// Keys of a sorted run that a later equal key supersedes, added to *dups.
template <typename K>
__global__ __launch_bounds__(256) void k_count_dups(const K* __restrict__ k, u64 n,
                                                    u32* __restrict__ dups) {
  constexpr u32 E = 16 / sizeof(K), U = 4;
  __shared__ u32 s_tmp[256 / 64 + 1];
  u32 c = 0;
  for (u64 base = (u64)blockIdx.x * 256 * E * U; base < n; base += (u64)gridDim.x * 256 * E * U) {
    KeyVec<K, (int)E> v[U];
    K nx[U];
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u64 i = base + ((u64)u * 256 + threadIdx.x) * E;
      if (i + E < n) {
        v[u] = *reinterpret_cast<const KeyVec<K, (int)E>*>(k + i);
        nx[u] = k[i + E];
      }
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u64 i = base + ((u64)u * 256 + threadIdx.x) * E;
      if (i + E < n) {
#pragma unroll
        for (u32 q = 0; q < E; ++q) c += v[u].k[q] == (q + 1 < E ? v[u].k[q + 1 < E ? q + 1 : q] : nx[u]);
      } else {
        for (u64 q = i; q + 1 < n && q < i + E; ++q) c += k[q] == k[q + 1];
      }
    }
  }
  u32 tot;
  block_exclusive_scan<256>(c, s_tmp, &tot);
  if (threadIdx.x == 0 && tot) atomicAdd(dups, tot);
}

// Any value equal to the reserved NOT_FOUND pattern -> *err = -1.
template <typename K>
__global__ void k_check_reserved(const K* __restrict__ v, u64 n, u32* __restrict__ err) {
  constexpr u32 E = 16 / sizeof(K);
  bool bad = false;
  // the caller's array may start anywhere its elements may
  const u64 head = ((16u - ((u64)v & 15u)) & 15u) / sizeof(K);
  const u64 lead = head < n ? head : n;
  const u64 words = (n - lead) / E;
  const u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x, nt = (u64)gridDim.x * blockDim.x;
  if (t < lead && v[t] == key_max<K>()) bad = true;
  for (u64 i = t; i < words; i += nt) {
    const KeyVec<K, (int)E> x = *reinterpret_cast<const KeyVec<K, (int)E>*>(v + lead + i * E);
#pragma unroll
    for (u32 q = 0; q < E; ++q) bad = bad || x.k[q] == key_max<K>();
  }
  for (u64 i = lead + words * E + t; i < n; i += nt) bad = bad || v[i] == key_max<K>();
  if (bad) atomicExch(err, 0xFFFFFFFFu);
}

// ---------------------------------------------------------------------------
// Initial build (Section 3.2): the n distinct sorted pairs are cut into
// groups of `fill` keys; group i becomes the single node of bucket i and its
// last key becomes maxBucket (MKBA[i]).  The last bucket's bound is KEY_MAX so
// that every key maps to a bucket.  Node i is the head of bucket i.
// ---------------------------------------------------------------------------
// V consecutive pairs per thread (V divides fill: one bucket and one 16-byte
// store each); the thread with a bucket's last pair writes its directory
// entry and header.  Bound by its 16 bytes of traffic per u32 pair:
// 2^26 pairs in 192 us (5.6 TB/s), the directory included (36 us as a kernel of
// its own, which read one key in 64).
template <typename K, u32 V>
__global__ __launch_bounds__(256) void k_build_nodes(const K* __restrict__ sk,
                                                     const K* __restrict__ sv, u64 n, u32 fill,
                                                     u32 cap, u32 nb, K* __restrict__ nkeys,
                                                     K* __restrict__ nvals, K* __restrict__ mkba,
                                                     NodeHdr* __restrict__ hdr,
                                                     u32* __restrict__ bnodes) {
  const u64 groups = (n + V - 1) / V;
  for (u64 g = (u64)blockIdx.x * 256 + threadIdx.x; g < groups; g += (u64)gridDim.x * 256) {
    const u64 i = g * V;
    const u32 b = (u32)(i / fill);
    const u32 s = (u32)(i - (u64)b * fill);
    const u64 at = (u64)b * cap + s;
    const u32 m = n - i < V ? (u32)(n - i) : V;
    K last;
    if (m == V) {
      const KeyVec<K, (int)V> k = *reinterpret_cast<const KeyVec<K, (int)V>*>(sk + i);
      const KeyVec<K, (int)V> v = *reinterpret_cast<const KeyVec<K, (int)V>*>(sv + i);
      *reinterpret_cast<KeyVec<K, (int)V>*>(nkeys + at) = k;
      *reinterpret_cast<KeyVec<K, (int)V>*>(nvals + at) = v;
      last = k.k[V - 1];
    } else {
      for (u32 q = 0; q < m; ++q) {
        nkeys[at + q] = sk[i + q];
        nvals[at + q] = sv[i + q];
      }
      last = sk[i + m - 1];
    }
    if (s + m == fill || i + m == n) {
      const K fence = b + 1 == nb ? key_max<K>() : last;
      mkba[b] = fence;
      NodeHdr h;
      h.fence = (u64)fence;
      h.size = s + m;
      h.next = kNil;
      hdr[b] = h;
      bnodes[b] = 1;
    }
  }
}

// The one empty bucket of a store without keys.
template <typename K>
__global__ void k_build_empty(K* __restrict__ mkba, NodeHdr* __restrict__ hdr,
                              u32* __restrict__ bnodes) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    mkba[0] = key_max<K>();
    NodeHdr h;
    h.fence = (u64)key_max<K>();
    h.size = 0;
    h.next = kNil;
    hdr[0] = h;
    bnodes[0] = 1;
  }
}

// Free stack holds every node id >= nb; Ctl counters reset; occupancy summary
// of nb buckets that all hold keys (none, when nkeys is 0).
__global__ void k_build_free(u32 nb, u32 pool, u64 nkeys, u32* __restrict__ free_ids,
                             Ctl* __restrict__ ctl, OccLevels occ) {
  u32 nfree = pool - nb;
  {
    const u64 n0 = occ_words0(nb), n1 = occ_words1(nb), n2 = occ_words2(nb);
    for (u64 w = (u64)blockIdx.x * blockDim.x + threadIdx.x; w < n0 + n1 + n2;
         w += (u64)gridDim.x * blockDim.x) {
      u64* const p = w < n0 ? occ.w0 + w : w < n0 + n1 ? occ.w1 + (w - n0) : occ.w2 + (w - n0 - n1);
      const u64 i = w < n0 ? w : w < n0 + n1 ? w - n0 : w - n0 - n1;
      const u64 below = w < n0 ? nb : w < n0 + n1 ? n0 : n1;   // what its level's bits stand for
      const u64 bits = below - i * 64;
      *p = nkeys == 0 ? 0ull : bits >= 64 ? ~0ull : (1ull << bits) - 1ull;
    }
  }
  for (u32 j = blockIdx.x * blockDim.x + threadIdx.x; j < nfree; j += gridDim.x * blockDim.x)
    free_ids[j] = pool - 1 - j;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->free_top = nfree;
    ctl->nkeys = nkeys;
    ctl->need = 0;
    ctl->call_err = 0;
    ctl->call_abort = 0;
    ctl->work_ovf = 0;
  }
}

// ---------------------------------------------------------------------------
// Dump: per-bucket totals (walking each chain), scan, then copy in key order.
// ---------------------------------------------------------------------------
__global__ void k_bucket_totals(const NodeHdr* __restrict__ hdr, u32 nb, u32 pool,
                                u32* __restrict__ tot) {
  for (u32 b = blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += gridDim.x * blockDim.x) {
    u32 t = 0;
    u32 node = b;
    u32 steps = 0;
    while (node < pool && steps++ < pool) {
      NodeHdr h = hdr[node];
      t += h.size;
      node = h.next;
    }
    tot[b] = t;
  }
}

// Exclusive scan of per-bucket totals: per-block partials, block-sum scan,
// add-back.  Used on the (non-hot) dump path.
__global__ __launch_bounds__(256) void k_scan_blocks_u32(const u32* __restrict__ in, u32 n,
                                                        u32* __restrict__ out,
                                                        u32* __restrict__ bsum) {
  __shared__ u32 s_tmp[256 / 64 + 1];
  u32 i = blockIdx.x * 256 + threadIdx.x;
  u32 v = i < n ? in[i] : 0u;
  u32 tot;
  u32 ex = block_exclusive_scan<256>(v, s_tmp, &tot);
  if (i < n) out[i] = ex;
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ void k_scan_addback(u32* __restrict__ out, u32 n, const u32* __restrict__ bsum) {
  u32 i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] += bsum[blockIdx.x];
}

// Runs of up to a node's keys in lanes i to i + 7 (c pairs from slot src on to
// position dst), copied by the whole wave.  All lanes of the wave call, i is
// uniform.
template <typename K>
__device__ __forceinline__ void wave_copy_eight(const ReadArgs<K>& a, u64 src, u64 dst, u32 c,
                                                u32 i) {
  constexpr u32 U = 8;
  bool more = true;
  for (u32 p = threadIdx.x & 63u; more; p += 64) {
    K k[U], v[U];
    more = false;
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u32 cu = wave_read(c, (int)(i + u));
      const u64 from = wave_read(src, (int)(i + u));
      if (p < cu) {
        k[u] = a.nkeys[from + p];
        v[u] = a.nvals[from + p];
      }
      more = more || cu > (p & ~63u) + 64;   // uniform
    }
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u64 to = wave_read(dst, (int)(i + u));
      if (p < wave_read(c, (int)(i + u))) {
        a.out_k[to + p] = k[u];
        a.out_v[to + p] = v[u];
      }
    }
  }
}

// A wave takes bpw (1 to 64) buckets, a lane each, and copies their nodes link by
// link: eight together (bpw <= 8), or, FLAT, as runs of one flattened list.  Chains
// that go on after kDumpLinks links, when they are few, are followed one by one,
// 64 links at a time.
constexpr u32 kDumpLinks = 4;
constexpr u32 kDumpFew = 4;

template <typename K, bool FLAT>
__global__ __launch_bounds__(256) void k_dump_copy(ReadArgs<K> a, const u32* __restrict__ off,
                                                   u64 out_cap, u32 bpw) {
  const u32 wave = (blockIdx.x * 256 + threadIdx.x) >> 6, nw = gridDim.x * 4u;
  const u32 lane = threadIdx.x & 63u;
  auto head = [&](u32 node) { return *reinterpret_cast<const u64*>(&a.hdr[node].size); };
  // pairs of a node to copy to position o
  auto count = [&](u64 w, u64 o) {
    const u32 sz = (u32)w < a.cap ? (u32)w : a.cap;
    const u64 room = o < out_cap ? out_cap - o : 0;
    return sz < room ? sz : (u32)room;
  };
  for (u64 b0 = (u64)wave * bpw; b0 < a.nb; b0 += (u64)nw * bpw) {
    const u64 b = b0 + lane;
    u32 node = lane < bpw && b < a.nb ? (u32)b : kNil;
    u64 o = node != kNil ? off[b] : 0;
    u32 steps = 0;   // nodes seen, the same for every chain still followed
    u64 m = wave_ballot(node < a.pool);
    while (m != 0 && (steps < kDumpLinks || (u32)__popcll(m) > kDumpFew)) {
      u32 c = 0, next = kNil;
      const u64 src = node < a.pool ? (u64)node * a.cap : 0;
      const u64 dst = o;
      ++steps;
      if (node < a.pool) {
        const u64 w = head(node);
        c = count(w, o);
        o += (u32)w < a.cap ? (u32)w : a.cap;
        next = steps < a.pool ? (u32)(w >> 32) : kNil;
      }
      if (FLAT) wave_copy_runs<K>(a, src, dst, c);
      else wave_copy_eight<K>(a, src, dst, c, 0);
      node = next;
      m = wave_ballot(node < a.pool);
    }
    for (; m; m &= m - 1) {
      const int l = (int)ctz64(m);
      u32 cur = wave_read(node, l);
      u64 at = wave_read(o, l);
      u32 seen = steps;
      while (cur < a.pool) {
        u64 src = 0, dst = 0;   // link i of this round in lane i
        u32 c = 0, n = 0;
        for (; n < 64 && cur < a.pool; ++n) {
          const u64 w = head(cur);
          if (lane == n) {
            src = (u64)cur * a.cap;
            dst = at;
            c = count(w, at);
          }
          at += (u32)w < a.cap ? (u32)w : a.cap;
          cur = ++seen < a.pool ? (u32)(w >> 32) : kNil;
        }
        for (u32 i = 0; i < n; i += 8) wave_copy_eight<K>(a, src, dst, c, i);
      }
    }
  }
}

// Nodes of at most 16 slots leave most lanes of a wave idle when they are copied
// one by one, so 64 of them go as one list (2^22 u32 keys in nodes of 8 slots: 150
// us against 185; of 16, 145 to 170 either way; of 32, 210).  Larger nodes go eight
// at a time (2^26 keys, 128 slots: 330 us against 400; 432 with a wave per bucket).
// In a store of few buckets a wave takes fewer, down to one, as long as the chip
// then has fewer than 32 waves per CU.
template <typename K>
void launch_dump_copy(const ReadArgs<K>& a, const u32* off, u64 out_cap, hipStream_t st) {
  const bool flat = a.cap <= 16;
  u32 bpw = 1;
  while (bpw < (flat ? 64u : 8u) && (u64)bpw * 8192u < a.nb) bpw <<= 1;
  const u32 per = 4 * bpw;
  const dim3 g(std::min<u32>((a.nb + per - 1) / per, 65535)), b(256);
  if (flat) hipLaunchKernelGGL((k_dump_copy<K, true>), g, b, 0, st, a, off, out_cap, bpw);
  else hipLaunchKernelGGL((k_dump_copy<K, false>), g, b, 0, st, a, off, out_cap, bpw);
}

// ---------------------------------------------------------------------------
// Device invariant checker.  err codes (first failure recorded):
//  1 key order inside a node      2 key outside its node's range
//  3 fence order along a chain    4 last fence != maxBucket
//  5 size > capacity              6 empty non-head node / empty head with next
//  7 chain length != bnodes       8 node id out of range / revisited
//  9 total keys != nkeys          10 live + free != pool
//  11 free id invalid or duplicated
// ---------------------------------------------------------------------------
template <typename K>
__global__ void k_check_buckets(const K* __restrict__ mkba, const NodeHdr* __restrict__ hdr,
                                const K* __restrict__ nkeys, const u32* __restrict__ bnodes,
                                u32 nb, u32 cap, u32 pool, u32* __restrict__ mark,
                                unsigned long long* __restrict__ counters,
                                u32* __restrict__ err) {
  for (u32 b = blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += gridDim.x * blockDim.x) {
    bool has_lo = b > 0;
    K lo = has_lo ? mkba[b - 1] : K(0);  // keys must be > lo (if has_lo)
    if (has_lo && !(mkba[b - 1] < mkba[b])) atomicCAS(err, 0u, 3u);
    u32 node = b;
    u32 len = 0;
    u64 keys = 0;
    bool first = true;
    K prev_fence = lo;
    bool have_prev = has_lo;
    while (node != kNil) {
      if (node >= pool) { atomicCAS(err, 0u, 8u); break; }
      if (atomicAdd(&mark[node], 1u) != 0u) { atomicCAS(err, 0u, 8u); break; }
      NodeHdr h = hdr[node];
      K fence = (K)h.fence;
      if (have_prev && !(prev_fence < fence)) atomicCAS(err, 0u, 3u);
      if (h.size > cap) { atomicCAS(err, 0u, 5u); break; }
      if (h.size == 0 && (!first || h.next != kNil)) atomicCAS(err, 0u, 6u);
      for (u32 s = 0; s < h.size; ++s) {
        K k = nkeys[(u64)node * cap + s];
        if (s > 0 && !(nkeys[(u64)node * cap + s - 1] < k)) atomicCAS(err, 0u, 1u);
        if ((have_prev && !(k > prev_fence)) || k > fence) atomicCAS(err, 0u, 2u);
      }
      keys += h.size;
      ++len;
      prev_fence = fence;
      have_prev = true;
      first = false;
      if (h.next == kNil && fence != mkba[b]) atomicCAS(err, 0u, 4u);
      node = h.next;
      if (len > pool) { atomicCAS(err, 0u, 8u); break; }
    }
    if (len != bnodes[b]) atomicCAS(err, 0u, 7u);
    atomicAdd(&counters[0], (unsigned long long)keys);
    atomicAdd(&counters[1], (unsigned long long)len);
  }
}

__global__ void k_check_free(const u32* __restrict__ free_ids, const Ctl* __restrict__ ctl,
                             u32 pool, u32* __restrict__ mark, u32* __restrict__ err) {
  u32 top = ctl->free_top;
  if (top > pool) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(err, 0u, 11u);
    return;
  }
  for (u32 j = blockIdx.x * blockDim.x + threadIdx.x; j < top; j += gridDim.x * blockDim.x) {
    u32 id = free_ids[j];
    if (id >= pool || atomicAdd(&mark[id], 1u) != 0u) atomicCAS(err, 0u, 11u);
  }
}

// ---------------------------------------------------------------------------
// Occupancy summary (flix_occ.hpp): invariant check.
// ---------------------------------------------------------------------------
// Invariant check: level 0 equals the head sizes, upper levels summarise the
// lower ones.  Records error 12 in *err.
__global__ void k_occ_check(const NodeHdr* __restrict__ hdr, u32 nb, OccLevels o,
                            u32* __restrict__ err) {
  const u64 n0 = occ_words0(nb), n1 = occ_words1(nb), n2 = occ_words2(nb);
  for (u64 w = (u64)blockIdx.x * blockDim.x + threadIdx.x; w < n0 + n1 + n2;
       w += (u64)gridDim.x * blockDim.x) {
    u64 want = 0, got;
    if (w < n0) {
      for (u32 i = 0; i < 64; ++i) {
        const u64 b = w * 64 + i;
        if (b < nb && hdr[b].size > 0) want |= 1ull << i;
      }
      got = o.w0[w];
    } else if (w < n0 + n1) {
      const u64 v = w - n0;
      for (u32 i = 0; i < 64; ++i)
        if (v * 64 + i < n0 && o.w0[v * 64 + i] != 0) want |= 1ull << i;
      got = o.w1[v];
    } else {
      const u64 v = w - n0 - n1;
      for (u32 i = 0; i < 64; ++i)
        if (v * 64 + i < n1 && o.w1[v * 64 + i] != 0) want |= 1ull << i;
      got = o.w2[v];
    }
    if (want != got) atomicCAS(err, 0u, 12u);
  }
}

}  // namespace flix
