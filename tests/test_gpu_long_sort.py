"""Long sorts (batches and loads above 2^22 items): exact stable permutation at
the edges of a tile, with all keys equal in some digits, and bulk loads with
and without superseded keys, into a pool with and without room to sort in."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import assert_same_contents, ktype, log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kb,n", [(32, (1 << 22) + 1), (32, 512 * 20 * 411 + 1), (32, 512 * 20 * 412 - 1),
                                  (64, 512 * 16 * 513), (64, 512 * 16 * 513 + 63)])
@pytest.mark.parametrize("shape", ["random", "few", "one_digit"])
def test_long_sort_is_the_stable_permutation(kb, n, shape):
    from paper_2604_16725_amd.flix import Store
    rng = np.random.default_rng(n + kb)
    k = rng.integers(0, 1 << kb, n, dtype=np.uint64).astype(ktype(kb))
    if shape == "few":
        k = k % ktype(kb)(1000)
    elif shape == "one_digit":
        k = (k & ktype(kb)(0xFF00)) | ktype(kb)(7)
    s = Store(key_bits=kb, capacity=64, max_batch=n)
    log(f"sort kb={kb} n={n} {shape}")
    ko, io = s.sort_pairs(to_dev(k))
    order = np.argsort(k, kind="stable")
    assert np.array_equal(to_host(io, 32), order.astype(np.uint32))
    assert np.array_equal(to_host(ko, kb), k[order])
    s.close()


@pytest.mark.parametrize("kb,n,distinct", [(32, (1 << 22) + 333, 0), (32, (1 << 22) + 333, 1 << 16),
                                           (64, 5_000_001, 0), (64, 5_000_001, 4_000_000),
                                           (32, 70001, 0), (32, 70001, 3000)])
@pytest.mark.parametrize("room", [True, False])
def test_bulk_load_duplicates_and_reload(kb, n, distinct, room):
    from oracle.oracle import Oracle
    from paper_2604_16725_amd.flix import FlixError, Store
    rng = np.random.default_rng(n + distinct + kb)
    cap = 32
    ks = w.KeySpace(kb, 21)
    base = ks.build(distinct or n)
    k = base if not distinct else base[rng.integers(0, distinct, n)]
    v = rng.integers(0, (1 << kb) - 1, n, dtype=np.uint64).astype(ktype(kb))
    nodes = -(-(distinct or n) // (cap // 2))
    node_bytes = cap * 2 * (kb // 8) + 16
    # without room: just the nodes the distinct keys need
    s = Store(key_bits=kb, capacity=cap, max_batch=1 << 12,
              pool_bytes=0 if room else nodes * node_bytes)
    o = Oracle(kb)
    for rep in range(2):   # the second load replaces contents that inserts have chained
        log(f"load kb={kb} n={n} distinct={distinct} room={room} rep={rep}")
        s.bulk_load(to_dev(k), to_dev(v))
        o.bulk_load(k, v)
        assert_same_contents(s, o, kb, f"load {rep}")
        bad = v.copy()
        bad[n // 2] = (1 << kb) - 1
        with pytest.raises(FlixError):
            s.bulk_load(to_dev(k), to_dev(bad))
        assert_same_contents(s, o, kb, "after a refused load")
        if room and rep == 0:
            run = (np.sort(base)[50] + np.arange(1, 2000)).astype(ktype(kb))
            s.insert(to_dev(run), to_dev(run))
            o.insert(run, run)
            assert_same_contents(s, o, kb, "chained")
    # a load that does not fit a fixed pool is refused and changes nothing
    if not room and not distinct:
        k2 = np.concatenate([k, ks.fresh(cap)])
        with pytest.raises(FlixError):
            s.bulk_load(to_dev(k2), to_dev(k2 >> ktype(kb)(1)))
        assert_same_contents(s, o, kb, "after a load that does not fit")
    s.close()
