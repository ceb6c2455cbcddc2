"""Contents in key order from every shape the copy distinguishes: nodes copied as
one list (up to 16 slots) or eight at a time, waves of one to 64 buckets, no
chain, short chains everywhere, few and many long chains in one wave, chains around
64 links.  Bit-exact against the oracle, with and without allocation."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import assert_same_contents, ktype, log, new_pair, to_dev, to_host

pytestmark = pytest.mark.gpu


def _check(s, o, kb):
    import torch
    assert_same_contents(s, o, kb)
    n = s.size()
    dt = torch.int32 if kb == 32 else torch.int64
    k, v = torch.zeros(n + 8, dtype=dt, device="cuda"), torch.zeros(n + 8, dtype=dt, device="cuda")
    assert s.dump_into(k, v, noalloc=True) == n
    ok, ov = o.dump()
    assert np.array_equal(to_host(k, kb)[:n], ok) and np.array_equal(to_host(v, kb)[:n], ov)
    assert not k[n:].any() and not v[n:].any()


# buckets: one wave, 1 to 8 per wave, and (nodes of 16 slots) 64 per wave
@pytest.mark.parametrize("kb,cap,buckets", [
    (32, 8, 1), (32, 8, 9000), (32, 16, 600000), (64, 16, 20000), (32, 32, 3), (64, 32, 70000),
    (32, 128, 8192), (32, 128, 8193), (64, 256, 300), (32, 256, 33000)])
def test_shapes(kb, cap, buckets):
    s, o = new_pair(kb, cap=cap, max_batch=1 << 18, fill=max(cap // 8, 1))
    fill = max(cap // 8, 1)
    n = (buckets - 1) * fill + 1
    k = np.sort(w.KeySpace(kb, 5).build(n))
    v = w.values_for(k, 6, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    log(f"kb={kb} cap={cap} buckets={buckets}")
    _check(s, o, kb)

    def insert(new):
        new = np.unique(new.astype(ktype(kb)))[: 1 << 18]
        nv = w.values_for(new, 7, kb)
        s.insert(to_dev(new), to_dev(nv))
        o.insert(new, nv)

    # chains of 3, 4, 5, 63, 66 and 130 or so nodes, some in neighbouring buckets
    for i, links in enumerate((3, 4, 5, 63, 66, 130)):
        at = k[min(n - 1, (n // 7) * (i + 1))]
        insert(at + np.arange(1, links * (cap // 2), dtype=np.uint64).astype(ktype(kb)))
    log("few chains")
    _check(s, o, kb)
    # twelve neighbouring buckets with chains of 20 nodes
    for i in range(12):
        at = k[min(n - 1, n // 2 + i * fill)]
        insert(at + np.arange(1, 20 * (cap // 2), dtype=np.uint64).astype(ktype(kb)))
    log("many chains in one wave")
    _check(s, o, kb)
    gone = o.dump()[0][::3][: 1 << 18]
    s.delete(to_dev(gone))
    o.delete(gone)
    log("after deletes")
    _check(s, o, kb)
    s.close()
