"""Ranges that go on past the nodes of their wave's other ranges: finished by the
whole wave, 64 nodes at a time.  Over plain buckets, chains shorter and longer than
64 nodes, stretches of empty buckets and the store's end, cut off or only counted;
few ranges (a wave each) and many with one long one among them; in calls and in a
drained queue.  Bit-exact against the sorted contents."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import ktype, log, new_pair, to_dev, to_host

pytestmark = pytest.mark.gpu


def _store(kb, cap, seed):
    rng = np.random.default_rng(seed)
    s, o = new_pair(kb, cap=cap, max_batch=1 << 17)
    ks = w.KeySpace(kb, seed)
    k = ks.build(120000)
    v = w.values_for(k, 2, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    order = np.sort(k)

    def both(new):
        nv = w.values_for(new, 3, kb)
        s.insert(to_dev(new), to_dev(nv))
        o.insert(new, nv)

    both(ks.fresh(50000))                                  # some short chains
    for at, links in ((1000, 3), (1500, 70), (1520, 64), (40000, 130), (119000, 20)):
        both(order[at] + np.arange(1, links * cap // 2).astype(ktype(kb)))
    gone = o.dump()[0][90000:130000]                       # hundreds of empty buckets
    s.delete(to_dev(gone))
    o.delete(gone)
    assert s.status() == 0 and s.check() == 0
    return s, o.dump(), rng


def _want(keys, lo, hi):
    a = np.searchsorted(keys, lo, "left")
    return a, np.where(lo <= hi, np.maximum(np.searchsorted(keys, hi, "right") - a, 0), 0)


@pytest.mark.parametrize("kb,cap", [(32, 8), (32, 64), (64, 16), (64, 128), (32, 256)])
def test_long_ranges(kb, cap):
    import torch
    s, (keys, vals), rng = _store(kb, cap, 7 + cap)
    n = keys.size
    top = ktype(kb)((1 << kb) - 1)
    shapes = [(1, n, n), (3, n, 1000), (5, 60000, 70000), (40, 9000, 9100), (300, 2000, 77),
              (5000, 300, 300), (70000, 3, 5), (100000, 40, 0)]
    for m, span, maxpq in shapes:
        first = rng.integers(0, n, m)
        last = np.minimum(first + rng.integers(0, span, m), n - 1)
        lo, hi = keys[first].copy(), keys[last].copy()
        lo[0], hi[0] = 0, top                              # the whole store
        hi[m // 2] = top                                   # to its end
        lo[m // 3] = keys[m // 3 % n] + ktype(kb)(1)       # between stored keys
        if m > 3:
            lo[3], hi[3] = top, 0
        first, count = _want(keys, lo, hi)
        if m * maxpq > 1 << 25:
            continue
        outs = [(True, True), (False, True), (True, False), (False, False)] if m < 100 else [(True, True)]
        for how in ("call", "drain"):
            for wk, wv in outs:
                if how == "drain" and not wv:
                    continue
                log(f"kb={kb} cap={cap} {how} {m} ranges of {span}, {maxpq} kept, keys {wk} values {wv}")
                size = max(m * maxpq, 1)
                dt = torch.int32 if kb == 32 else torch.int64
                ok = torch.zeros(size, dtype=dt, device="cuda") if wk else None
                ov = torch.zeros(size, dtype=dt, device="cuda") if wv else None
                c = torch.zeros(m, dtype=torch.int32, device="cuda")
                if how == "call":
                    s.range(to_dev(lo), to_dev(hi), maxpq, counts=c, out_k=ok, out_v=ov,
                            want_keys=wk, want_vals=wv)
                else:
                    s.drain([dict(op="range", keys=to_dev(lo), aux=to_dev(hi), counts=c, out_k=ok,
                                  out_v=ov, max_per_query=maxpq)])
                got = c.cpu().numpy().view(np.uint32)
                bad = np.nonzero(got != count)[0]
                assert bad.size == 0, (bad[:5], got[bad[:3]], count[bad[:3]])
                kept = np.minimum(count, maxpq)
                row = np.repeat(np.arange(m), kept)
                at = np.arange(row.size) - np.repeat(np.cumsum(kept) - kept, kept)
                for t, x in ((ok, keys), (ov, vals)):
                    if t is not None and maxpq:
                        a = to_host(t, kb)
                        assert np.array_equal(a[row * maxpq + at], x[first[row] + at])
                        a = a.copy()
                        a[row * maxpq + at] = 0
                        assert not a.any()                 # nothing else was written
    assert s.status() == 0
    s.close()
