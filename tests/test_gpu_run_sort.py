"""Sort of batches between the short form and the long one: the exact stable
permutation whatever the keys (evenly spread, dense stretches, repeated keys,
the ends of the key range) at the edges of tiles, of the run length and of the
form's range, and the payloads of updates through it."""
import numpy as np
import pytest
import torch

from paper_2604_16725_amd import workloads as w
from paper_2604_16725_amd.flix import Store
from tests.gpu_helpers import assert_same_contents, ktype, log, new_pair, to_dev, to_host

pytestmark = pytest.mark.gpu

LIMIT = 7168 * 256
SIZES = [1, 2047, 2049, 8192, 8193, 12289, 65537, 300001, (1 << 20) + 1, LIMIT, LIMIT + 1]


def _shapes(rng, kb, n):
    top = (1 << kb) - 1
    t = ktype(kb)
    even = rng.integers(0, top, n, dtype=np.uint64, endpoint=True).astype(t)
    yield "even", even
    yield "sequence", rng.permutation(n).astype(t)
    # a span just above a power of two, far from 0
    yield "span", (even % t((1 << (kb - 6)) + 5) + t(1 << (kb - 2))).astype(t)
    starts = rng.integers(0, top - n, 16, dtype=np.uint64)
    yield "stretches", (starts[rng.integers(0, 16, n)] +
                        rng.integers(0, n // 16 + 1, n).astype(np.uint64)).astype(t)
    yield "hot", np.where(rng.random(n) < 0.7, t(12345), even)
    yield "ends", np.where(rng.random(n) < 0.5, t(0), t(top))
    yield "equal", np.full(n, top // 3, dtype=np.uint64).astype(t)
    few = rng.integers(0, top, 5, dtype=np.uint64).astype(t)
    yield "few", few[rng.integers(0, 5, n)]


@pytest.mark.parametrize("kb", [32, 64])
def test_exact_permutation(kb):
    rng = np.random.default_rng(kb)
    s = Store(key_bits=kb, max_batch=max(SIZES))
    for n in SIZES:
        for name, k in _shapes(rng, kb, n):
            log(f"kb={kb} n={n} {name}")
            ko, io = s.sort_pairs(to_dev(k))
            perm = np.argsort(k, kind="stable")
            assert np.array_equal(to_host(io, 32), perm.astype(np.uint32)), (n, name)
            assert np.array_equal(to_host(ko, kb), k[perm]), (n, name)
    assert s.status() == 0
    s.close()


@pytest.mark.parametrize("kb", [32, 64])
def test_updates_keep_the_last_value(kb):
    n = 40000
    rng = np.random.default_rng(kb + 1)
    s, o = new_pair(kb, max_batch=n)
    ks = w.KeySpace(kb, 7)
    base = ks.build(30000)
    v = w.values_for(base, 5, kb)
    s.bulk_load(to_dev(base), to_dev(v))
    o.bulk_load(base, v)
    fresh = ks.fresh(n)
    stretch = (np.sort(base)[1000] + np.arange(1, 12001).astype(ktype(kb))).astype(ktype(kb))
    for name, k in [("fresh", fresh),
                    ("hot", np.where(rng.random(n) < 0.7, fresh[0], fresh)),
                    ("stretch", stretch[rng.integers(0, stretch.size, n)])]:
        log(f"kb={kb} {name}")
        nv = rng.integers(0, (1 << kb) - 1, n, dtype=np.uint64).astype(ktype(kb))
        for _ in range(2):   # the second call finds the first one's counters
            s.insert(to_dev(k), to_dev(nv))
            o.insert(k, nv)
        assert_same_contents(s, o, kb, f"{name} inserted")
        d = np.concatenate([k[: n // 2], ks.absent(n - n // 2)])
        s.delete(to_dev(d))
        o.delete(d)
        assert_same_contents(s, o, kb, f"{name} deleted")
    assert s.status() == 0
    s.close()


def test_sort_on_two_streams():
    """Two stores' sorts of long runs at once: each ends whatever the other holds."""
    n = 1 << 19
    rng = np.random.default_rng(9)
    k = np.where(rng.random(n) < 0.6, np.uint64(99), rng.integers(0, 1 << 63, n, dtype=np.uint64))
    perm = np.argsort(k, kind="stable").astype(np.uint32)
    stores = [Store(key_bits=64, max_batch=n) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    d = to_dev(k)
    torch.cuda.synchronize()
    out = []
    for _ in range(4):
        for s, st in zip(stores, streams):
            with torch.cuda.stream(st):
                out.append(s.sort_pairs(d))
    torch.cuda.synchronize()
    for ko, io in out:
        assert np.array_equal(to_host(io, 32), perm)
        assert np.array_equal(to_host(ko, 64), k[perm])
    for s in stores:
        assert s.status() == 0
        s.close()
