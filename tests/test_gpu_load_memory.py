"""Bulk loads that run out of memory part way: an allocator hook refuses the
n-th allocation of a load, alone or with all that follow.  The load succeeds, or
it returns FLIX_ENOMEM and the store holds its old contents, is empty, or refuses
every call until a load succeeds; a batch of the old size still sorts."""
import ctypes

import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import assert_same_contents, log, to_dev, to_host

pytestmark = pytest.mark.gpu


class _Hook:
    """Device memory from torch's caching allocator, refused where told to."""

    def __enter__(self):
        import torch
        from paper_2604_16725_amd import flix
        self.lib = flix.load_library()
        self.fail = lambda i: False
        self.count = 0
        self.live = set()

        def alloc(nbytes, ctx):
            i, self.count = self.count, self.count + 1
            if self.fail(i):
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device())
            self.live.add(p)
            return p

        def free(ptr, ctx):
            self.live.remove(ptr)
            torch.cuda.caching_allocator_delete(ptr)

        self.fns = (flix._ALLOC_FN(alloc), flix._FREE_FN(free))
        rc = self.lib.flix_set_allocator(*[ctypes.cast(f, ctypes.c_void_p) for f in self.fns], None)
        assert rc == 0
        return self

    def refuse(self, fail):
        self.count = 0
        self.fail = fail

    def __exit__(self, *exc):
        self.lib.flix_set_allocator(None, None, None)


def _refused(fn):
    from paper_2604_16725_amd.flix import FLIX_ENOMEM, FlixError
    try:
        fn()
    except FlixError as e:
        assert e.code == FLIX_ENOMEM, e
        return True
    return False


# the load that runs out: larger than what is stored (sort scratch, directory and
# pool grow), smaller (the pool shrinks), with duplicates (the pool changes its size
# twice), into a new store, after loads with duplicates (temporary buffers first)
@pytest.mark.parametrize("kb,n0,n1,dup,loads", [
    (32, 20000, 150000, 1, 1), (64, 90000, 3000, 1, 1), (32, 50000, 120000, 5, 1),
    (64, 0, 40000, 1, 0), (64, 20000, 90000, 3, 3), (32, 60000, 100000, 2, 3)])
@pytest.mark.parametrize("rest", [False, True])
def test_refused_allocations(kb, n0, n1, dup, loads, rest):
    import torch
    from oracle.oracle import Oracle
    from paper_2604_16725_amd.flix import DrainGraph, Store
    ka = w.KeySpace(kb, 1).build(max(n0, 1))[:n0]
    va = w.values_for(ka, 2, kb)
    kn = np.tile(w.KeySpace(kb, 3).build(n1 // dup), dup)
    vn = w.values_for(kn, 4, kb) ^ np.arange(kn.size).astype(kn.dtype) % 64
    probe = np.concatenate([kn[:500], ka[:500]])
    new, old = Oracle(kb), Oracle(kb)
    new.bulk_load(kn, vn)
    old.bulk_load(ka, va)
    outcomes = set()
    with _Hook() as hook:
        for i in range(40):
            hook.refuse(lambda j: False)
            s = Store(key_bits=kb, capacity=64, max_batch=1 << 15)
            for _ in range(loads):
                twice = 2 if loads > 1 else 1
                s.bulk_load(to_dev(np.tile(ka, twice)), to_dev(np.tile(va, twice)))
            out = torch.zeros(probe.size, dtype=s.dtype, device="cuda")
            st = torch.cuda.Stream()
            dprobe = to_dev(probe)
            g = DrainGraph(s, [dict(op="lookup", keys=dprobe, out_v=out)], stream=st)
            hook.refuse((lambda j: j >= i) if rest else (lambda j: j == i))
            failed = _refused(lambda: s.bulk_load(to_dev(kn), to_dev(vn)))
            asked = hook.count
            hook.refuse(lambda j: False)
            log(f"kb={kb} {n0}->{n1} dup={dup} after {loads} refuse {'from ' if rest else ''}{i}: failed={failed}")
            if not failed:
                outcomes.add("loaded")
                assert_same_contents(s, new, kb)
            elif _refused(lambda: s.lookup(to_dev(probe))):
                outcomes.add("refuses")
                kd, vd = to_dev(kn[:100]), to_dev(vn[:100])
                for fn in (lambda: s.insert(kd, vd), lambda: s.delete(kd), lambda: s.successor(kd),
                           lambda: s.range(kd, kd, 1), s.size, s.dump, s.stats, s.restructure,
                           lambda: s.drain([dict(op="delete", keys=kd)])):
                    assert _refused(fn)
                assert s.check() == -2 and s.status() == 0
                g.launch(stream=st)
                torch.cuda.synchronize()
                assert s.status() == -5
            else:
                left = old if s.size() else Oracle(kb)
                outcomes.add("kept" if s.size() else "empty")
                assert_same_contents(s, left, kb)
                assert np.array_equal(to_host(s.lookup(to_dev(probe)), kb), left.lookup(probe))
                more = w.KeySpace(kb, 9).build(30000)   # the old batch size still sorts
                s.insert(to_dev(more), to_dev(w.values_for(more, 5, kb)))
                assert s.status() == 0 and s.size() >= 30000
            s.bulk_load(to_dev(kn), to_dev(vn))
            assert_same_contents(s, new, kb)
            g.launch(stream=st)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(out, kb), new.lookup(probe)) and s.status() == 0
            g.close()
            s.close()
            assert not hook.live
            if not failed and i >= asked:
                break
        else:
            raise AssertionError("the load never ran out of allocations to refuse")
    log(outcomes)
    assert "loaded" in outcomes and len(outcomes) > (1 if rest else 0)


def test_fixed_pool_too_small_keeps_the_contents():
    from oracle.oracle import Oracle
    from paper_2604_16725_amd.flix import Store
    k = w.KeySpace(32, 1).build(4000)
    v = w.values_for(k, 2, 32)
    big = w.KeySpace(32, 5).build(60000)
    s = Store(key_bits=32, capacity=64, max_batch=1 << 12, pool_bytes=528 * 400)
    o = Oracle(32)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    assert _refused(lambda: s.bulk_load(to_dev(big), to_dev(w.values_for(big, 3, 32))))
    assert_same_contents(s, o, 32)
    s.close()


@pytest.mark.parametrize("kb", [32, 64])
def test_loads_with_and_without_duplicates_in_turn(kb):
    """The pool ends at the size a fresh store's would, whatever was loaded before."""
    from oracle.oracle import Oracle
    from paper_2604_16725_amd.flix import Store
    s = Store(key_bits=kb, capacity=64, max_batch=1 << 12)
    for i, (n, dup) in enumerate([(60000, 4), (60000, 4), (60000, 4), (60000, 4), (60000, 1),
                                  (60000, 1), (60000, 2), (60000, 3), (60000, 2), (60000, 1),
                                  (9000, 3), (9000, 3), (0, 1), (60000, 4)]):
        k = np.tile(w.KeySpace(kb, 3 + i).build(max(n // dup, 1)), dup)[:n]
        v = w.values_for(k, 4, kb) ^ np.arange(k.size).astype(k.dtype) % 64
        log(f"kb={kb} n={n} dup={dup}")
        o = Oracle(kb)
        o.bulk_load(k, v)
        fresh = Store(key_bits=kb, capacity=64, max_batch=1 << 12)
        for x in (s, fresh):
            x.bulk_load(to_dev(k), to_dev(v))
            assert_same_contents(x, o, kb)
        assert s.stats() == fresh.stats()
        fresh.close()
    s.close()
