"""Read batches long enough for the flipped form (sort, merge-path shares, buckets
resolve their slices), over both key widths, every operation, the lane and capacity
shapes of its kernel, and over chains, emptied buckets and shrunken nodes: equal to
the same queries answered in parts short enough for the input-order form, and those
on a sample to the oracle.  An epoch whose read lists are that long, too."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import check_reads, ktype, log, new_pair, to_dev, to_host

pytestmark = pytest.mark.gpu

POINT = {32: 3 << 21, 64: 1 << 24}     # longest batches answered in input order
RANGE = 1 << 24


def _grown(kb, cap, lanes, max_batch, seed, n=60000):
    rng = np.random.default_rng(seed)
    s, o = new_pair(kb, cap=cap, lanes=lanes, max_batch=max_batch)
    ks = w.KeySpace(kb, seed)
    k = ks.build(n)

    def both(new):
        nv = w.values_for(new, 3, kb)
        s.insert(to_dev(new), to_dev(nv))
        o.insert(new, nv)

    v = w.values_for(k, 2, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    order = np.sort(k)
    both(ks.fresh(n // 2))
    for at, links in ((n // 9, 5), (n // 5, 40)):              # chains
        both(order[at] + np.arange(1, links * max(cap // 2, 8)).astype(ktype(kb)))
    gone = o.dump()[0]
    gone = np.concatenate([gone[n // 2: n // 2 + n // 5], gone[: n // 9: 3]])
    s.delete(to_dev(gone))                                     # empty buckets, shrunken nodes
    o.delete(gone)
    assert s.status() == 0
    return s, o, rng


def _queries(o, rng, n, kb):
    """On the GPU: stored keys and their neighbours, uniform keys, both ends."""
    import torch
    keys = to_dev(o.dump()[0])
    g = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))
    at = torch.randint(0, keys.numel(), (n,), generator=g, device="cuda")
    q = keys[at] + torch.randint(-1, 2, (n,), generator=g, device="cuda").to(keys.dtype)
    u = torch.randint(-(1 << (kb - 1)), (1 << (kb - 1)) - 1, (n // 5,), generator=g, device="cuda")
    q[: n // 5] = u.to(keys.dtype)
    q[-1], q[-2] = -1, 0
    return q.contiguous()


def _parts(n, limit):
    return [slice(i, min(i + limit // 2, n)) for i in range(0, n, limit // 2)]


def _check(s, q, op, limit, maxpq=2, width=None):
    import torch
    n = q.numel()
    assert n > limit
    if op == "range":
        hi = q + width
        c, k, v = s.range(q, hi, maxpq)
        for p in _parts(n, limit):
            pc, pk, pv = s.range(q[p].contiguous(), hi[p].contiguous(), maxpq)
            assert torch.equal(c[p], pc)
            live = torch.arange(maxpq, device="cuda")[None, :] < pc[:, None]
            assert not (pc < 0).any()
            for whole, part in ((k, pk), (v, pv)):
                a, b = whole.view(n, maxpq)[p], part.view(-1, maxpq)
                assert torch.equal(a[live], b[live])
        return
    got = getattr(s, op)(q)
    got = got if isinstance(got, tuple) else (got,)
    for p in _parts(n, limit):
        part = getattr(s, op)(q[p].contiguous())
        part = part if isinstance(part, tuple) else (part,)
        for a, b in zip(got, part):
            assert torch.equal(a[p], b), op


# every instantiation of the resolving kernel (lanes, keys per lane)
@pytest.mark.parametrize("kb,cap,lanes", [
    (32, 8, 16), (32, 16, 16), (32, 32, 16), (32, 64, 16), (32, 128, 16), (32, 256, 16),
    (32, 32, 32), (32, 64, 32), (32, 128, 32), (32, 256, 32), (32, 64, 64), (32, 128, 64),
    (32, 256, 64)])
def test_point_reads_32(kb, cap, lanes):
    limit = POINT[kb]
    n = limit + 4097
    s, o, rng = _grown(kb, cap, lanes, n, cap + lanes)
    q = _queries(o, rng, n, kb)
    check_reads(s, o, kb, to_host(q[n // 2: n // 2 + 3000].contiguous(), kb), maxpq=4)
    for op in ("lookup", "successor", "predecessor"):
        log(f"kb={kb} cap={cap} lanes={lanes} {op} n={n}")
        _check(s, q, op, limit)
    assert s.status() == 0
    s.close()


@pytest.mark.parametrize("kb,cap,lanes", [(64, 8, 16), (64, 32, 16), (64, 128, 16), (64, 256, 16),
                                          (64, 64, 32), (64, 256, 32), (64, 128, 64), (64, 256, 64)])
def test_point_reads_64(kb, cap, lanes):
    limit = POINT[kb]
    n = limit + 1023
    s, o, rng = _grown(kb, cap, lanes, n, cap + lanes)
    q = _queries(o, rng, n, kb)
    check_reads(s, o, kb, to_host(q[n // 2: n // 2 + 3000].contiguous(), kb), maxpq=4)
    for op in ("lookup", "successor", "predecessor"):
        log(f"kb={kb} cap={cap} lanes={lanes} {op} n={n}")
        _check(s, q, op, limit)
    assert s.status() == 0
    s.close()


@pytest.mark.parametrize("kb,cap,lanes", [(32, 16, 16), (32, 128, 16), (32, 256, 32), (32, 64, 64),
                                          (64, 16, 16), (64, 128, 16), (64, 64, 32), (64, 256, 64)])
def test_ranges(kb, cap, lanes):
    n = RANGE + 77
    s, o, rng = _grown(kb, cap, lanes, n, cap + lanes)
    q = _queries(o, rng, n, kb)
    # about three stored keys per range, and longer ones in the chains
    width = (1 << kb) // 60000 * 3
    log(f"kb={kb} cap={cap} lanes={lanes} ranges n={n}")
    _check(s, q, "range", RANGE, maxpq=2, width=width)
    assert s.status() == 0
    s.close()


@pytest.mark.parametrize("kb", [32, 64])
def test_epoch_with_long_read_lists(kb):
    import torch
    n = RANGE + 5
    s, o, rng = _grown(kb, 64, 16, n, 3)
    q = _queries(o, rng, n, kb)
    hi = q + (1 << kb) // 60000 * 2
    uk = w.KeySpace(kb, 3).build(60000)[:20000]
    uv = w.values_for(uk, 8, kb)
    uv[::2] = np.array((1 << kb) - 1, dtype=np.uint64).astype(ktype(kb))
    out = torch.zeros(n, dtype=q.dtype, device="cuda")
    c = torch.zeros(n, dtype=torch.int32, device="cuda")
    rk, rv = torch.zeros_like(out), torch.zeros_like(out)
    want = torch.cat([s.lookup(q[p].contiguous()) for p in _parts(n, POINT[kb])])
    wc, wk = [], []
    for p in _parts(n, RANGE):
        a, b, _ = s.range(q[p].contiguous(), hi[p].contiguous(), 1)
        wc.append(a)
        wk.append(b)
    wc, wk = torch.cat(wc), torch.cat(wk)
    duk, duv = to_dev(uk), to_dev(uv)
    log(f"kb={kb} epoch with {n} lookups and ranges")
    e = s.make_epoch(lookup_keys=q, lookup_vals=out, range_lo=q, range_hi=hi, range_max=1,
                     range_counts=c, range_keys=rk, range_vals=rv, update_keys=duk, update_vals=duv)
    s.epoch_prepare(0, e)
    s.epoch_apply(0, e)
    assert s.status() == 0
    assert torch.equal(out, want) and torch.equal(c, wc)
    some = wc > 0
    assert torch.equal(rk[some], wk[some])
    dele = uv == np.array((1 << kb) - 1, dtype=np.uint64).astype(ktype(kb))
    o.delete(uk[dele])
    o.insert(uk[~dele], uv[~dele])
    got_k, got_v = s.dump()
    ok, ov = o.dump()
    assert np.array_equal(to_host(got_k, kb), ok) and np.array_equal(to_host(got_v, kb), ov)
    s.close()
