"""Reads in input order (one lane per query, directory searched as a tree):
bit-exact against the oracle where the tree gains a level, at the edges of
waves and workgroups, for every node capacity, over chained, empty and
shrunken buckets, and for ranges of every length."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import assert_same_contents, check_reads, ktype, log, new_pair, to_dev

pytestmark = pytest.mark.gpu


def _queries(rng, kb, keys, n):
    """Stored keys, their neighbours, uniform keys and both ends of the key space."""
    k = keys[rng.integers(0, keys.size, n)] if keys.size else np.zeros(n, ktype(kb))
    u = w.perm(rng.integers(0, 1 << 31, n, dtype=np.uint64), 77, kb)
    q = np.where(rng.random(n) < 0.4, u, k + rng.integers(0, 3, n).astype(ktype(kb)) - ktype(kb)(1))
    q[: min(n, 2)] = [0, (1 << kb) - 1][: min(n, 2)]
    return q.astype(ktype(kb))


# buckets (fill 1..cap/2) around the top level's 4096 (u32) / 2048 (u64)
# entries and around 16 times that
@pytest.mark.parametrize("kb,cap,fill,buckets", [
    (32, 8, 1, 1), (32, 8, 1, 4095), (32, 8, 1, 4096), (32, 8, 1, 4097), (32, 16, 1, 65536),
    (32, 32, 2, 65537), (64, 8, 1, 2047), (64, 8, 1, 2049), (64, 16, 1, 32768), (64, 32, 3, 32769),
    (32, 64, 32, 300), (32, 128, 64, 300), (32, 128, 128, 300), (32, 256, 128, 300),
    (64, 64, 32, 300), (64, 128, 64, 300), (64, 256, 255, 300)])
def test_directory_levels_and_node_shapes(kb, cap, fill, buckets):
    rng = np.random.default_rng(1000 * kb + cap + buckets)
    s, o = new_pair(kb, cap=cap, max_batch=1 << 16, fill=fill)
    n = (buckets - 1) * fill + 1
    k = w.KeySpace(kb, 5).build(n)
    v = w.values_for(k, 6, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    for m in (1, 3, 63, 64, 65, 255, 256, 257, 5001):
        log(f"kb={kb} cap={cap} fill={fill} buckets={buckets} m={m}")
        check_reads(s, o, kb, _queries(rng, kb, k, m), maxpq=5, where=f"m={m}")
    s.close()


@pytest.mark.parametrize("kb,cap", [(32, 8), (32, 64), (32, 256), (64, 8), (64, 128)])
def test_chains_gaps_and_empty_store(kb, cap):
    rng = np.random.default_rng(kb + cap)
    s, o = new_pair(kb, cap=cap, max_batch=1 << 16)
    log(f"empty store kb={kb} cap={cap}")
    check_reads(s, o, kb, _queries(rng, kb, np.zeros(0, ktype(kb)), 130), where="empty")
    ks = w.KeySpace(kb, 9)
    k = ks.build(20000)
    v = w.values_for(k, 2, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    # a dense run (chains), growth everywhere, then a gap of emptied buckets
    run = (np.sort(k)[1000] + np.arange(1, 4000)).astype(ktype(kb))
    for new in (run, ks.fresh(30000)):
        nv = w.values_for(new, 3, kb)
        s.insert(to_dev(new), to_dev(nv))
        o.insert(new, nv)
    present = np.concatenate([k, run])
    log(f"chains kb={kb} cap={cap}")
    check_reads(s, o, kb, _queries(rng, kb, present, 4097), where="chains")
    gone = np.sort(o.dump()[0])[5000:30000]
    s.delete(to_dev(gone))
    o.delete(gone)
    log(f"gap kb={kb} cap={cap}")
    check_reads(s, o, kb, _queries(rng, kb, gone, 4097), where="gap")
    assert_same_contents(s, o, kb)
    s.close()


@pytest.mark.parametrize("kb,m,span,maxpq", [
    (32, 1, 30000, 30000), (32, 70, 300, 300), (32, 70, 300, 7), (64, 40000, 17, 17),
    (32, 40000, 1, 1), (64, 500, 64, 0), (64, 9000, 130, 128)])
def test_range_lengths(kb, m, span, maxpq):
    rng = np.random.default_rng(m + span)
    s, o = new_pair(kb, cap=64, max_batch=1 << 16)
    k = w.KeySpace(kb, 11).build(40000)
    v = w.values_for(k, 12, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    order = np.sort(k)
    first = rng.integers(0, k.size, m)
    first[0] = 0
    lo = order[first]
    hi = order[np.minimum(first + rng.integers(0, span + 1, m), k.size - 1)]
    hi[-1] = order[-1]
    if m > 8:
        lo[3], hi[3] = hi[3], lo[3]            # mostly an empty interval
        lo[5], hi[5] = 0, (1 << kb) - 1        # the whole store
    log(f"ranges kb={kb} m={m} span={span} maxpq={maxpq}")
    check_reads(s, o, kb, lo, maxpq=maxpq, lo=lo, hi=hi, where="ranges")
    s.close()


@pytest.mark.parametrize("kb,cap,fill", [(32, 64, 64), (32, 256, 256), (32, 32, 31), (64, 64, 63),
                                         (64, 256, 255), (64, 128, 128)])
def test_keys_far_from_where_they_are_looked_for(kb, cap, fill):
    """Nodes whose keys crowd at either end, lie in clumps or are spread evenly:
    the first block looked at is right, next to the right one or far off."""
    rng = np.random.default_rng(cap + fill + kb)
    half = np.uint64(1) << np.uint64(kb - 10)
    i = np.arange(fill, dtype=np.uint64)
    bits = np.uint64(kb - 12)
    grow = np.unique(np.concatenate([np.uint64(1) << (i % bits), i]))[:fill]
    shapes = [i, half - i - np.uint64(1), grow, half - np.uint64(1) - grow[::-1],
              i * (half // np.uint64(fill)), (i % np.uint64(3)) * (half // np.uint64(4)) + i]
    k = np.unique(np.concatenate([np.uint64(1 + b) * half + np.uint64(5) + shapes[b % 6]
                                  for b in range(300)])).astype(ktype(kb))
    v = w.values_for(k, 6, kb)
    s, o = new_pair(kb, cap=cap, max_batch=1 << 16, fill=fill)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    for q in (k, k - ktype(kb)(1), k + ktype(kb)(1), _queries(rng, kb, k, 20011)):
        log(f"kb={kb} cap={cap} fill={fill} n={q.size}")
        check_reads(s, o, kb, q[: 1 << 16], maxpq=5)
    d = k[rng.random(k.size) < 0.6]
    s.delete(to_dev(d[: 1 << 16]))
    o.delete(d[: 1 << 16])
    check_reads(s, o, kb, _queries(rng, kb, k, 20011), maxpq=5, where="shrunken")
    s.close()


@pytest.mark.parametrize("n", [(3 << 21) - 1, 3 << 21, (3 << 21) + 1])
def test_long_batches_either_side_of_the_rule(n):
    rng = np.random.default_rng(n)
    s, _ = new_pair(32, cap=32, max_batch=n)
    k = np.unique(rng.integers(1, (1 << 32) - 2, 100000, dtype=np.uint64)).astype(np.uint32)
    v = w.values_for(k, 6, 32)
    s.bulk_load(to_dev(k), to_dev(v))
    q = rng.integers(0, (1 << 32) - 2, n, dtype=np.uint64).astype(np.uint32)
    q[::3] = k[rng.integers(0, k.size, q[::3].size)]
    at = np.searchsorted(k, q)
    ok = at < k.size
    succ = np.where(ok, k[np.minimum(at, k.size - 1)], np.uint32(0xFFFFFFFF))
    val = np.where(ok, v[np.minimum(at, k.size - 1)], np.uint32(0xFFFFFFFF))
    dq = to_dev(q)
    log(f"n={n}")
    sk, sv = s.successor(dq)
    assert np.array_equal(sk.cpu().numpy().view(np.uint32), succ)
    assert np.array_equal(sv.cpu().numpy().view(np.uint32), val)
    got = s.lookup(dq).cpu().numpy().view(np.uint32)
    assert np.array_equal(got, np.where(succ == q, val, np.uint32(0xFFFFFFFF)))
    s.close()
