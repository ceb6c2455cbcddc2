// The persistent drain kernel (flix_drain.hpp) in a translation unit of its
// own, instantiated for both key widths, both digit widths and every lane-group
// width of its update phases.
#include <algorithm>

#include "flix_launch.hpp"

namespace flix {
namespace {

template <typename K, int RB, int GL>
hipError_t drain_t(const DrainLaunch& d, hipStream_t st) {
  size_t shm = DrainSmemSize<K, RB>::fixed();
  const size_t upd = (size_t)(256 / GL) * 2 * d.lds_items * sizeof(K);
  if (upd > shm) shm = upd;
  auto kfn = k_drain<K, RB, GL>;
  hipError_t e;
  if (*d.grid == 0 || *d.shm != shm) {
    if (shm > 65536 &&
        (e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm)) != hipSuccess)
      return e;
    int per_cu = 0, dev = 0, cus = 0;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kfn, 256, shm)) != hipSuccess ||
        (e = hipGetDevice(&dev)) != hipSuccess ||
        (e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
      return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    // At most two workgroups per CU: updates pay several grid barriers, whose
    // cost grows with the arrivals, reads gain from more waves.  A queue of 40
    // mixed batches (flix_drain.hpp) takes 1.47 ms with one, 1.50 with two, 1.67
    // with three; two were best on the longer mixed-batch stream while reads were
    // sorted and paid barriers, too (540 Mops/s; one 537, three 475).
    *d.grid = std::min(per_cu, 2) * cus;
    *d.shm = shm;
  }
  DrainArgs<K> a;
  a.batches = d.batches;
  a.nbatch = d.nbatch;
  a.layout = d.layout;
  a.cap = d.cap;
  a.ctl = d.ctl;
  a.bk[0] = (K*)d.bk[0];
  a.bk[1] = (K*)d.bk[1];
  a.bp[0] = d.bp[0];
  a.bp[1] = d.bp[1];
  a.hist = d.hist;
  a.status = d.status;
  a.status_cl = d.status_cl;
  a.status_words = d.status_words;
  a.cluster_words = d.cluster_words;
  a.work = d.work;
  a.lds_items = d.lds_items;
  a.chunk = d.chunk;
  a.dctl = d.dctl;
  a.tstamp = d.tstamp;
  a.max_batch = d.max_batch;
  hipLaunchKernelGGL(kfn, dim3(*d.grid), dim3(256), shm, st, a);
  return hipGetLastError();
}

template <typename K, int RB>
hipError_t drain_rb(const DrainLaunch& d, hipStream_t st) {
  switch (d.gl) {
    case 16: return drain_t<K, RB, 16>(d, st);
    case 32: return drain_t<K, RB, 32>(d, st);
    default: return drain_t<K, RB, 64>(d, st);
  }
}

}  // namespace

hipError_t drain_launch(const DrainLaunch& d, hipStream_t st) {
  if (d.key_bits == 32)
    return d.radix_bits == 4 ? drain_rb<u32, 4>(d, st) : drain_rb<u32, 8>(d, st);
  return d.radix_bits == 4 ? drain_rb<u64, 4>(d, st) : drain_rb<u64, 8>(d, st);
}

}  // namespace flix
