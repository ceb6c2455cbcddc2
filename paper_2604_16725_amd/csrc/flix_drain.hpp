// Persistent fused drain: one co-resident grid executes a whole queue of
// mixed-type batches (lookup, successor, range, insert, delete) in order.
// Read batches are answered in input order by the searches of flix_direct.hpp
// and run into one another: the grid meets at a barrier before a read batch
// only where its buffers overlap those of a batch since the last barrier.
// Update batches run in phases with a grid barrier between them instead of a
// kernel boundary: short ones sort by counting, slices, update kernel; longer ones
// histogram, onesweep passes, slices, update kernel.  The queue lives in device
// memory, so one launch (or one hipGraph replay) drains it, and the batches can
// change between replays.
//
// What bounds it: a barrier of the grid costs 11 to 20 us (the release of each
// workgroup writes its XCD's L2 back).  While every batch was sorted, with
// P + 3 barriers, 40 batches of 2^8 to 2^20 operations on 2^26 keys (4.9 M
// reads, eight updates of 0.5 k to 49 k keys) took 8.7 ms; they take 1.5 ms.
// Eight updates of 12,288 u32 keys take 0.78 ms, of 12,289 1.63 (u64 0.86, 2.49):
// the limit of the short form is that of the calls, not where a drain would have it.
//
// Ordering and memory: a grid barrier is arrive (agent-scope release +
// atomic) / wait (generation word) / agent-scope acquire.  Tiles of a pass are
// walked in increasing order by every workgroup, so a tile only waits on
// tiles that are resident or finished.  Look-back words carry an epoch from
// a device counter that every drain advances, so nothing is cleared between
// passes, drains or graph replays.
#pragma once

#include "flix_device.hpp"
#include "flix_direct.hpp"
#include "flix_small.hpp"
#include "flix_sort.hpp"
#include "flix_update.hpp"

namespace flix {

constexpr u32 kOpInsert = 3;
constexpr u32 kOpDelete = 4;
constexpr u32 kOpLast = 5;   // predecessor

struct alignas(16) DrainBatch {
  u32 op;
  u32 n;
  u32 maxpq;
  u32 reserved;
  const void* keys;   // keys (range: lo)
  const void* aux;    // insert: values; range: hi
  void* out_v;
  void* out_k;
  u32* counts;
  void* reserved2;
};

// Arrival groups of the grid barrier: workgroup b arrives on counter b % 8,
// which matches the round-robin placement of workgroups on the 8 XCDs, so no
// counter takes more than an eighth of the arrivals.
constexpr u32 kBarGroups = 8;

struct DrainCtl {
  u32 bar_gen;       // barrier generation
  u32 epoch;         // last look-back epoch used by a drain
  u32 err;           // sticky: 1 barrier wait or look-back gave up, 4 bad descriptor
  u32 top_count;     // groups complete at the current barrier
  u32 pad0[28];
  u32 grp[kBarGroups][32];   // arrivals per group, one 128-byte line each
};

// The store's layout as the kernels see it.  Bulk loads reallocate the
// directory and the pool, so a drain captured in a graph must not hold these
// pointers: it reads this record, which every bulk load rewrites, when each
// replay starts.
struct alignas(16) StoreLayout {
  const void* mkba;
  NodeHdr* hdr;
  void* nkeys;
  void* nvals;
  u32* bnodes;
  u32* free_ids;
  u32 nb;
  u32 pool;
  u32 pad[2];
  OccLevels occ;
  const void* dir;   // search levels above mkba (flix_direct.hpp)
  const void* pad2;
};

template <typename K>
struct DrainArgs {
  const DrainBatch* batches;
  u32 nbatch;
  // store: layout read from device memory at kernel start
  const StoreLayout* layout;
  u32 cap;
  Ctl* ctl;
  // scratch
  K* bk[2];
  void* bp[2];
  u32* hist;          // [2][P*R]
  u64* status;
  u64* status_cl;
  u64 status_words;
  u64 cluster_words;
  WorkItem* work;
  u32 lds_items;
  u32 chunk;
  DrainCtl* dctl;
  unsigned long long* tstamp;   // [nbatch + 1]: start, then one per batch (may be null)
  u32 max_batch;
};

// Grid-wide barrier for a co-resident grid.  Each workgroup publishes its
// writes (agent-scope release fence: the L2 of its XCD is written back),
// arrives on its group counter; the last arrival of a group arrives on the
// top counter, and the last group flips the generation.  Waiters poll the
// generation with relaxed loads and invalidate their caches once, after the
// flip (an acquire load per poll would invalidate the L2 on every poll).
// Bounded: a workgroup that waits too long records an error.  Returns true
// (in every thread of the workgroup) once the grid has failed, a barrier wait
// or a sort look-back having given up: the caller must then leave the kernel,
// since later phases would read buffers that earlier phases did not finish.
__device__ __forceinline__ bool grid_sync(DrainCtl* c, u32 nblocks) {
  __shared__ u32 s_abort;
  __syncthreads();
  if (threadIdx.x == 0) {
    const u32 g = blockIdx.x % kBarGroups;
    const u32 members = (nblocks - g + kBarGroups - 1) / kBarGroups;
    const u32 ngroups = nblocks < kBarGroups ? nblocks : kBarGroups;
    const u32 gen = __hip_atomic_load(&c->bar_gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // this workgroup's writes
    bool flipped = false;
    const u32 a = __hip_atomic_fetch_add(&c->grp[g][0], 1u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) + 1u;
    if (a == members) {
      __hip_atomic_store(&c->grp[g][0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");   // the group's writes, onward
      const u32 t = __hip_atomic_fetch_add(&c->top_count, 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT) + 1u;
      if (t == ngroups) {
        __hip_atomic_store(&c->top_count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        __hip_atomic_store(&c->bar_gen, gen + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        flipped = true;
      }
    }
    if (!flipped) {
      // Bounded wait; once any barrier has failed (the grid was not fully
      // resident) no later barrier waits, so the kernel ends promptly.
      u32 polls = 0;
      while (__hip_atomic_load(&c->bar_gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gen) {
        if (__hip_atomic_load(&c->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u) break;
        if (++polls > (1u << 22)) {
          atomicOr(&c->err, 1u);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // everyone's writes
    s_abort = __hip_atomic_load(&c->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u;
  }
  __syncthreads();
  return s_abort != 0;
}

template <typename K, int RB>
struct DrainSmemSize {
  static constexpr size_t hist = sizeof(HistSmem<K, RB>);
  static constexpr size_t pass_val = sizeof(OnesweepSmem<K, K, RB, kDrainSortNT, kDrainSortIPT, kPayValue>);
  static constexpr size_t pass_none = sizeof(OnesweepSmem<K, u32, RB, kDrainSortNT, kDrainSortIPT, kPayNone>);
  static constexpr size_t slices = sizeof(SliceSmem<K, (sizeof(K) == 4 ? 1024 : 512), 256>);
  static constexpr size_t fixed() {
    size_t m = hist;
    m = m > pass_val ? m : pass_val;
    m = m > pass_none ? m : pass_none;
    m = m > slices ? m : slices;
    m = m > sizeof(RankSmem<K>) ? m : sizeof(RankSmem<K>);
    m = m > sizeof(SliceUnitSmem) ? m : sizeof(SliceUnitSmem);
    return m;
  }
};

// Memory a batch reads and writes outside the store, as [begin, end) pairs.
struct BatchSpans {
  u64 in[2][2];
  u64 out[3][2];
};
template <typename K>
__device__ __forceinline__ BatchSpans batch_spans(const DrainBatch& d, u32 max_batch) {
  BatchSpans s;
  const u64 n = (d.n > max_batch || d.op > kOpLast) ? 0 : d.n;
  const bool range = d.op == kOpRange;
  const u64 pairs = range ? n * d.maxpq : n;
  const bool outs = n != 0 && d.op != kOpInsert && d.op != kOpDelete;
  const bool keyed = range || d.op == kOpSuccessor || d.op == kOpPredecessor;
  auto put = [](u64 (&r)[2], const void* p, u64 bytes) {
    r[0] = (u64)p;
    r[1] = p ? (u64)p + bytes : 0;
  };
  put(s.in[0], n ? d.keys : nullptr, n * sizeof(K));
  put(s.in[1], n && (range || d.op == kOpInsert) ? d.aux : nullptr, n * sizeof(K));
  put(s.out[0], outs ? d.out_v : nullptr, pairs * sizeof(K));
  put(s.out[1], outs && keyed ? d.out_k : nullptr, pairs * sizeof(K));
  put(s.out[2], outs && range ? d.counts : nullptr, n * sizeof(u32));
  return s;
}
__device__ __forceinline__ bool spans_conflict(const BatchSpans& a, const BatchSpans& b) {
  bool c = false;
  auto meet = [](const u64 (&x)[2], const u64 (&y)[2]) { return x[0] < y[1] && y[0] < x[1]; };
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int k = 0; k < 3; ++k) c = c || meet(a.out[i], b.out[k]);
#pragma unroll
    for (int k = 0; k < 2; ++k) c = c || meet(a.out[i], b.in[k]) || meet(a.in[k], b.out[i]);
  }
  return c;
}
// Time stamp of a wave's part of a batch, taken when its answers are stored: its
// stores are counted by vmcnt, which a release within the workgroup does not wait
// for.  (An agent-scope release would, but writes the XCD's L2 back: 11 us and
// more.)
__device__ __forceinline__ void stamp_stored(unsigned long long* at) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // no store sinks below
  __builtin_amdgcn_s_waitcnt(0);
  if ((threadIdx.x & 63u) == 0) atomicMax(at, (unsigned long long)wall_clock64());
}

// answers_over_keys of a batch (false for an update).
template <typename K>
__device__ __forceinline__ bool batch_over_keys(const DrainBatch& d, u32 max_batch) {
  const BatchSpans s = batch_spans<K>(d, max_batch);
  const bool range = d.op == kOpRange;
  bool c = false;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    c = c || ((range || s.out[i][0] != s.in[0][0]) && s.out[i][0] < s.in[0][1] &&
              s.in[0][0] < s.out[i][1]);
  return c;
}

// Read batch of a drain: units of Q * qpw queries (Q of each lane) go to the
// waves of the grid in turn, from wave `rot` on.  Returns whether this wave had any.
template <typename K, int OP, int Q>
__device__ __forceinline__ bool drain_read(const ReadArgs<K>& ra, const DirTree<K>& tree,
                                           const K* s_top, u32 wave, u32 waves, u32 rot,
                                           u32 qpw) {
  const u32 lane = threadIdx.x & 63u;
  const u32 units = (ra.m + qpw * Q - 1) / (qpw * Q);
  bool any = false;
  for (u32 u = wave >= rot ? wave - rot : wave + waves - rot; u < units; u += waves) {
    u32 j[Q];
    bool live[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      j[q] = (u * Q + q) * qpw + lane;
      live[q] = lane < qpw && j[q] < ra.m;
    }
    direct_read<K, OP, Q>(ra, tree, s_top, j, live);
    any = true;
  }
  return any;
}

template <typename K, int RB, int GL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_drain(DrainArgs<K> a) {
  extern __shared__ unsigned char smem[];
  __shared__ UpdShared s_upd;
  __shared__ u32 s_epoch;
  __shared__ __align__(16) K s_top[DirTop<K>::n];
  constexpr int R = RadixShape<K, RB>::R;
  constexpr int P = RadixShape<K, RB>::P;
  // queries per lane in flight: the registers of the update phases leave the
  // grid two or three waves per SIMD, so a wave has to bring its own
  // parallelism
  constexpr int Q = sizeof(K) == 4 ? 4 : 2;
  constexpr int SS = sizeof(K) == 4 ? 1024 : 512;  // slice share
  const u32 G = gridDim.x;
  const u32 blk = blockIdx.x;
  DrainCtl* dc = a.dctl;
  const StoreLayout L = *a.layout;
  const K* const mkba = (const K*)L.mkba;
  K* const nkeys = (K*)L.nkeys;
  K* const nvals = (K*)L.nvals;
  if (L.nb == 0) {   // a replay after a bulk load that left the store without a pool
    if (blk == 0 && threadIdx.x == 0) atomicOr(&dc->err, 4u);
    return;
  }
  const DirTree<K> tree = dir_tree<K>(mkba, (const K*)L.dir, L.nb);
  load_top<K, 256>(tree, s_top);
  const u32 waves = G * 4u;
  const u32 wave = (threadIdx.x >> 6) * G + blk;   // neighbouring units on different CUs

  // Epochs: every workgroup reads the base before anyone advances it (the
  // advance happens after the first barrier, by the most this drain can use,
  // so a drain that stops early never leaves epochs to be reused).  Near
  // wrap-around the status words are cleared first.
  if (threadIdx.x == 0) s_epoch = __hip_atomic_load(&dc->epoch, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  u32 epoch = s_epoch;
  const u32 need_epochs = a.nbatch * (u32)P + 1u;
  if (epoch + need_epochs >= (1u << 30) - 1u) {
    for (u64 i = (u64)blk * 256 + threadIdx.x; i < a.status_words; i += (u64)G * 256) a.status[i] = 0;
    for (u64 i = (u64)blk * 256 + threadIdx.x; i < a.cluster_words; i += (u64)G * 256)
      a.status_cl[i] = 0;
    epoch = 0;
  }
  // both histogram slots start at zero
  if (blk == 0)
    for (int i = threadIdx.x; i < 2 * P * R; i += 256) a.hist[i] = 0;
  if (a.tstamp)
    for (u64 i = (u64)blk * 256 + threadIdx.x; i <= a.nbatch; i += (u64)G * 256)
      a.tstamp[i] = i == 0 ? wall_clock64() : 0ull;
  const u32 epoch_end = epoch + need_epochs;
  const bool failed0 = grid_sync(dc, G);
  if (blk == 0 && threadIdx.x == 0)
    __hip_atomic_store(&dc->epoch, epoch_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (failed0) return;

  u32 nz = 0;     // update batches processed so far: selects the histogram slot
  u32 rot = 0;    // wave that takes the next read unit
  u32 pend = 0;   // first batch since the last barrier
  u64 over = 0;   // of 64 batches: which answer over keys still to be read
  for (u32 bi = 0; bi < a.nbatch; ++bi) {
    if ((bi & 63u) == 0) {
      // (a lane each: tested batch by batch, 40 mixed batches of up to 3700 u32 keys
      // took 628 us, so 601)
      const u32 l = bi + (threadIdx.x & 63u);
      over = wave_ballot(l < a.nbatch && batch_over_keys<K>(a.batches[l], a.max_batch));
    }
    const DrainBatch d = a.batches[bi];   // uniform
    const u32 n = d.n;
    if (n > a.max_batch || d.op > kOpLast) {   // rewritten descriptor out of range
      if (blk == 0 && threadIdx.x == 0) atomicOr(&dc->err, 4u);
      continue;
    }
    if (n == 0) {
      if (blk == 0 && threadIdx.x == 0 && a.tstamp)
        atomicMax(&a.tstamp[bi + 1], (unsigned long long)wall_clock64());
      continue;
    }
    const bool is_update = d.op == kOpInsert || d.op == kOpDelete;
    // Read batches run into one another: a barrier comes before a batch only
    // where it reads what a batch since the last barrier writes, or writes
    // what one reads or writes.  One lane compares with each of those batches
    // (at most 64).
    {
      const u32 npend = bi - pend;
      bool wait = npend >= 64u;
      if (!wait && npend > 0) {
        const u32 lane = threadIdx.x & 63u;
        bool c = false;
        if (lane < npend)
          c = spans_conflict(batch_spans<K>(a.batches[pend + lane], a.max_batch),
                             batch_spans<K>(d, a.max_batch));
        wait = wave_ballot(c) != 0;
      }
      if (wait) {
        if (grid_sync(dc, G)) return;
        pend = bi;
      }
    }
    if (!is_update) {
      const bool copied = (over >> (bi & 63u)) & 1u;
      if (copied) {   // to the sort's scratch, which no batch since the last barrier uses
        for (u32 i = blk * 256 + threadIdx.x; i < n; i += G * 256) a.bk[0][i] = ((const K*)d.keys)[i];
        if (grid_sync(dc, G)) return;
      }
      ReadArgs<K> ra;
      ra.skeys = copied ? a.bk[0] : (const K*)d.keys;
      ra.sidx = nullptr;
      ra.m = n;
      ra.mkba = mkba;
      ra.nb = L.nb;
      ra.hdr = L.hdr;
      ra.nkeys = nkeys;
      ra.nvals = nvals;
      ra.cap = a.cap;
      ra.share = 0;
      ra.out_v = (K*)d.out_v;
      ra.out_k = (K*)d.out_k;
      ra.hi = (const K*)d.aux;
      ra.counts = d.counts;
      ra.maxpq = d.maxpq;
      ra.pool = L.pool;
      ra.err = &a.ctl->status;
      ra.occ = L.occ.w0;
      ra.cuts = nullptr;
      bool any;
      u32 per = 64 * Q;
      switch (d.op) {
        case kOpLookup:
          any = drain_read<K, kOpLookup, Q>(ra, tree, s_top, wave, waves, rot, 64);
          break;
        case kOpSuccessor:
          any = drain_read<K, kOpSuccessor, Q>(ra, tree, s_top, wave, waves, rot, 64);
          break;
        case kOpRange:
          per = range_queries_per_wave(64, n, waves);
          any = drain_read<K, kOpRange, 1>(ra, tree, s_top, wave, waves, rot, per);
          break;
        default:
          any = drain_read<K, kOpPredecessor, Q>(ra, tree, s_top, wave, waves, rot, 64);
          break;
      }
      rot = (u32)((rot + (n + per - 1) / per) % waves);
      if (any && a.tstamp) stamp_stored(&a.tstamp[bi + 1]);   // the last wave's time stays
      if (copied) {   // the scratch is free for the next batch
        if (grid_sync(dc, G)) return;
        pend = bi + 1;
      }
      continue;
    }
    if (n <= kSmallMax) {
      // short update: sort by counting, work items, apply
      const bool ins = d.op == kOpInsert;
      for (u32 u = blk; u * kRankKeys < n; u += G) {
        __syncthreads();
        rank_unit<K>((const K*)d.keys, ins ? (const K*)d.aux : nullptr, n, u, a.bk[0],
                     (K*)a.bp[0], *reinterpret_cast<RankSmem<K>*>(smem));
      }
      if (grid_sync(dc, G)) return;
      SliceArgs<K> sa;
      sa.skeys = a.bk[0];
      sa.svals = ins ? (const K*)a.bp[0] : nullptr;
      sa.m = n;
      sa.mkba = mkba;
      sa.nb = L.nb;
      sa.hdr = L.hdr;
      sa.bnodes = L.bnodes;
      sa.cap = a.cap;
      sa.share = 0;
      sa.work = a.work;
      sa.rcap = 0;
      sa.ctl = a.ctl;
      sa.parts = a.ctl->part;
      const u32 units = (n + kSliceKeys - 1) / kSliceKeys;
      SliceUnitSmem& su = *reinterpret_cast<SliceUnitSmem*>(smem);
      for (u32 u = blk; u < units; u += G) {
        if (threadIdx.x == 0) su.bad = 0;
        __syncthreads();
        if (ins) slice_unit<K, true>(sa, tree, s_top, u, su);
        else slice_unit<K, false>(sa, tree, s_top, u, su);
      }
      if (grid_sync(dc, G)) return;
      UpdArgs<K> ua;
      ua.mkba = mkba;
      ua.skeys = a.bk[0];
      ua.svals = sa.svals;
      ua.m = n;
      ua.hdr = L.hdr;
      ua.nkeys = nkeys;
      ua.nvals = nvals;
      ua.bnodes = L.bnodes;
      ua.free_ids = L.free_ids;
      ua.cap = a.cap;
      ua.chunk = a.chunk;
      ua.pool = L.pool;
      ua.work = a.work;
      ua.rcap = 0;
      ua.ctl = a.ctl;
      ua.status = &a.ctl->status;
      ua.occ = L.occ;
      ua.parts = a.ctl->part;
      ua.nparts = ins ? units : 0u;
      if (ins) insert_items<K, GL, 256, true>(ua, a.lds_items, blk, G, smem, s_upd);
      else delete_items<K, GL, 256, true>(ua, a.lds_items, blk, G, smem, s_upd);
      if (grid_sync(dc, G)) return;
      pend = bi + 1;
      if (blk == 0 && threadIdx.x == 0 && a.tstamp)
        atomicMax(&a.tstamp[bi + 1], (unsigned long long)wall_clock64());
      continue;
    }
    const u32 slot = nz & 1u;
    ++nz;
    u32* hist = a.hist + slot * (P * R);
    if (blk == 0) {
      if (threadIdx.x == 0) {
        a.ctl->need = 0;
        a.ctl->call_err = 0;
        a.ctl->call_abort = 0;
      }
      reset_work_regions(a.ctl, threadIdx.x);
    }
    // ---- histogram
    radix_hist_part<K, RB>((const K*)d.keys, n, hist, blk, G,
                           *reinterpret_cast<HistSmem<K, RB>*>(smem));
    if (grid_sync(dc, G)) return;
    // ---- onesweep passes
    const u32 ntiles = (n + kSortTile - 1) / kSortTile;
    for (int p = 0; p < P; ++p) {
      ++epoch;
      // constant indices only: a runtime index into the argument arrays
      // would move them to scratch memory
      K* const bk0 = a.bk[0];
      K* const bk1 = a.bk[1];
      void* const bp0 = a.bp[0];
      void* const bp1 = a.bp[1];
      const K* ki = (p == 0) ? (const K*)d.keys : ((p & 1) ? bk0 : bk1);
      K* ko = (p & 1) ? bk1 : bk0;
      if (d.op == kOpInsert) {
        PassArgs<K, K> pa;
        pa.kin = ki;
        pa.vin = (p == 0) ? (const K*)d.aux : (const K*)((p & 1) ? bp0 : bp1);
        pa.kout = ko;
        pa.vout = (K*)((p & 1) ? bp1 : bp0);
        pa.n = n; pa.shift = (u32)(p * RB); pa.hist_p = hist + p * R;
        pa.status = a.status; pa.status_cl = a.status_cl; pa.epoch = epoch; pa.err = &dc->err;
        for (u32 t = blk; t < ntiles; t += G)
          onesweep_tile<K, K, RB, kDrainSortNT, kDrainSortIPT, kPayValue>(
              pa, t, *reinterpret_cast<OnesweepSmem<K, K, RB, kDrainSortNT, kDrainSortIPT, kPayValue>*>(smem));
      } else if (d.op == kOpDelete) {
        PassArgs<K, u32> pa;
        pa.kin = ki; pa.vin = nullptr; pa.kout = ko; pa.vout = nullptr;
        pa.n = n; pa.shift = (u32)(p * RB); pa.hist_p = hist + p * R;
        pa.status = a.status; pa.status_cl = a.status_cl; pa.epoch = epoch; pa.err = &dc->err;
        for (u32 t = blk; t < ntiles; t += G)
          onesweep_tile<K, u32, RB, kDrainSortNT, kDrainSortIPT, kPayNone>(
              pa, t, *reinterpret_cast<OnesweepSmem<K, u32, RB, kDrainSortNT, kDrainSortIPT, kPayNone>*>(smem));
      }
      if (grid_sync(dc, G)) return;
    }
    const int r = ((P - 1) & 1) ? 1 : 0;
    // the other histogram slot was last used by the previous batch and is
    // next used by the following one, after at least one more barrier
    if (blk == 0)
      for (int i = threadIdx.x; i < P * R; i += 256) a.hist[(slot ^ 1u) * (P * R) + i] = 0;
    // ---- apply
    {
      SliceArgs<K> sa;
      sa.skeys = a.bk[r];
      sa.svals = d.op == kOpInsert ? (const K*)a.bp[r] : nullptr;
      sa.m = n;
      sa.mkba = mkba;
      sa.nb = L.nb;
      sa.hdr = L.hdr;
      sa.bnodes = L.bnodes;
      sa.cap = a.cap;
      sa.share = SS;
      sa.work = a.work;
      sa.rcap = work_region_cap(a.max_batch);
      sa.ctl = a.ctl;
      const u32 nshares = (u32)(((u64)n + L.nb + SS - 1) / SS);
      for (u32 vb = blk; vb < nshares; vb += G) {
        if (d.op == kOpInsert)
          slices_share<K, 256, SS, true>(sa, vb, *reinterpret_cast<SliceSmem<K, SS, 256>*>(smem));
        else
          slices_share<K, 256, SS, false>(sa, vb, *reinterpret_cast<SliceSmem<K, SS, 256>*>(smem));
      }
      if (grid_sync(dc, G)) return;
      UpdArgs<K> ua;
      ua.mkba = mkba;
      ua.skeys = a.bk[r];
      ua.svals = d.op == kOpInsert ? (const K*)a.bp[r] : nullptr;
      ua.m = n;
      ua.hdr = L.hdr;
      ua.nkeys = nkeys;
      ua.nvals = nvals;
      ua.bnodes = L.bnodes;
      ua.free_ids = L.free_ids;
      ua.cap = a.cap;
      ua.chunk = a.chunk;
      ua.pool = L.pool;
      ua.work = a.work;
      ua.rcap = work_region_cap(a.max_batch);
      ua.ctl = a.ctl;
      ua.status = &a.ctl->status;
      ua.occ = L.occ;
      if (d.op == kOpInsert)
        insert_items<K, GL, 256, false>(ua, a.lds_items, blk, G, smem, s_upd);
      else
        delete_items<K, GL, 256, false>(ua, a.lds_items, blk, G, smem, s_upd);
    }
    if (grid_sync(dc, G)) return;
    pend = bi + 1;
    if (blk == 0 && threadIdx.x == 0 && a.tstamp) atomicMax(&a.tstamp[bi + 1], (unsigned long long)wall_clock64());
  }
  if (a.tstamp) {
    // the stamps of overlapping batches in batch order: running maximum
    if (grid_sync(dc, G)) return;
    if (blk == 0 && threadIdx.x < 64) {
      unsigned long long run = 0;
      for (u32 i0 = 0; i0 <= a.nbatch; i0 += 64) {
        const u32 i = i0 + threadIdx.x;
        u64 v = i <= a.nbatch ? ld_agent((const u64*)&a.tstamp[i]) : 0ull;
#pragma unroll
        for (u32 o = 1; o < 64; o <<= 1) {
          const u64 y = shfl64(v, threadIdx.x >= o ? threadIdx.x - o : threadIdx.x);
          if (threadIdx.x >= o) v = v > y ? v : y;
        }
        v = v > run ? v : run;
        run = shfl64(v, 63);
        if (i <= a.nbatch) a.tstamp[i] = v;
      }
    }
  }
}

}  // namespace flix
