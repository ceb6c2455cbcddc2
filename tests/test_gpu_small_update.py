"""Short update batches (sorted by counting, work items by directory search):
contents equal the oracle's at the edges of the ranking and slice units and of
the form's range, with repeated keys, slices that cross units, chains, and
batches that must be rejected as a whole; through inserts and deletes, epochs
and drained queues."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import assert_same_contents, ktype, log, new_pair, to_dev

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 31, 33, 255, 256, 511, 2049, 4097, 12287, 12288, 12289]


def _batches(rng, kb, base, ks, n):
    """New keys; mostly repeated keys; one dense run; stored keys."""
    yield "new", ks.fresh(n)
    pool = np.concatenate([base[:50], ks.fresh(50)])
    yield "repeated", pool[rng.integers(0, pool.size, n)]
    start = np.sort(base)[base.size // 3]
    run = (start + np.arange(1, n + 1).astype(ktype(kb))).astype(ktype(kb))
    yield "run", rng.permutation(run)
    yield "stored", base[rng.integers(0, base.size, n)]


@pytest.mark.parametrize("kb,cap,lanes", [(32, 8, 16), (32, 128, 16), (32, 64, 64), (64, 128, 32),
                                          (64, 32, 16)])
def test_insert_and_delete_sizes(kb, cap, lanes):
    rng = np.random.default_rng(kb + cap)
    s, o = new_pair(kb, cap=cap, lanes=lanes, max_batch=1 << 15)
    ks = w.KeySpace(kb, 31)
    base = ks.build(60000)
    v = w.values_for(base, 5, kb)
    s.bulk_load(to_dev(base), to_dev(v))
    o.bulk_load(base, v)
    for n in SIZES:
        for name, k in _batches(rng, kb, base, ks, n):
            log(f"kb={kb} cap={cap} n={n} {name}")
            nv = rng.integers(0, (1 << kb) - 1, n, dtype=np.uint64).astype(ktype(kb))
            s.insert(to_dev(k), to_dev(nv))
            o.insert(k, nv)
            d = np.concatenate([k[: n // 2], ks.absent(n - n // 2)])
            rng.shuffle(d)
            s.delete(to_dev(d))
            o.delete(d)
        assert s.status() == 0
        assert_same_contents(s, o, kb, f"n={n}")
    s.close()


@pytest.mark.parametrize("kb", [32, 64])
def test_rejected_batches_change_nothing(kb):
    cap, f = 16, 8
    ks = w.KeySpace(kb, 41)
    base = ks.build(4000)
    v = w.values_for(base, 5, kb)
    nodes = -(-4000 // f) + 40
    s, o = new_pair(kb, cap=cap, max_batch=1 << 14, pool_bytes=nodes * (cap * 2 * (kb // 8) + 16))
    s.bulk_load(to_dev(base), to_dev(v))
    o.bulk_load(base, v)
    log("reserved value in a short batch")
    k = ks.fresh(700)
    bad = w.values_for(k, 6, kb)
    bad[433] = (1 << kb) - 1
    s.insert(to_dev(k), to_dev(bad), check=False)
    assert s.status() == -1
    assert_same_contents(s, o, kb, "after a reserved value")
    log("more new nodes than the pool holds")
    k = ks.fresh(12000)
    s.insert(to_dev(k), to_dev(w.values_for(k, 7, kb)), check=False)
    assert s.status() == -2
    assert_same_contents(s, o, kb, "after an exhausted pool")
    log("repeated keys count once: as many operations, few nodes")
    k = ks.fresh(30)[np.arange(3000) % 30]
    nv = w.values_for(k, 8, kb)
    s.insert(to_dev(k), to_dev(nv))
    o.insert(k, nv)
    assert s.status() == 0
    assert_same_contents(s, o, kb, "after repeated keys")
    s.close()


@pytest.mark.parametrize("kb,n", [(32, 3), (64, 300), (32, 5000), (64, 12288), (64, 12289)])
def test_epochs_and_drains(kb, n):
    import torch
    rng = np.random.default_rng(kb + n)
    dt = torch.int32 if kb == 32 else torch.int64
    s, o = new_pair(kb, cap=64, max_batch=1 << 14)
    ks = w.KeySpace(kb, 51)
    base = ks.build(50000)
    v = w.values_for(base, 5, kb)
    s.bulk_load(to_dev(base), to_dev(v))
    o.bulk_load(base, v)
    gone = ktype(kb)((1 << kb) - 1)
    for rep in range(3):
        log(f"epoch kb={kb} n={n} rep={rep}")
        pool = np.concatenate([base[rng.integers(0, base.size, n)], ks.fresh(n)])
        uk = pool[rng.integers(0, pool.size, n)]
        uv = w.values_for(uk, 60 + rep, kb)
        uv[rng.random(n) < (0.5, 0.0, 1.0)[rep]] = gone
        q = pool[rng.integers(0, pool.size, 777)]
        out = torch.zeros(777, dtype=dt, device="cuda")
        dq, duk, duv = to_dev(q), to_dev(uk), to_dev(uv)
        ep = s.make_epoch(lookup_keys=dq, lookup_vals=out, update_keys=duk, update_vals=duv)
        s.epoch_prepare(rep % 2, ep)
        dq.zero_()             # the lookups were taken by the prepare
        s.epoch_apply(rep % 2, ep)
        want = o.lookup(q)
        last = {int(a): b for a, b in zip(uk, uv)}
        dk = np.array([a for a, b in last.items() if b == gone], ktype(kb))
        ik = np.array([a for a, b in last.items() if b != gone], ktype(kb))
        iv = np.array([b for b in last.values() if b != gone], ktype(kb))
        if dk.size:
            o.delete(dk)
        if ik.size:
            o.insert(ik, iv)
        assert s.status() == 0
        assert np.array_equal(out.cpu().numpy().view(ktype(kb)), want)
        assert_same_contents(s, o, kb, f"epoch {rep}")
    log(f"drain kb={kb} n={n}")
    qs = []
    for i in range(6):
        k = np.concatenate([base[rng.integers(0, base.size, n // 2)], ks.fresh(n - n // 2)])
        iv = w.values_for(k, 70 + i, kb)
        d = k[rng.integers(0, n, n)]
        qs += [dict(op="insert", keys=to_dev(k), aux=to_dev(iv)), dict(op="delete", keys=to_dev(d))]
        o.insert(k, iv)
        o.delete(d)
    s.drain(qs)
    assert s.status() == 0
    assert_same_contents(s, o, kb, "drained")
    s.close()
