"""Answers stored over the keys they answer: at any distance between the two
buffers the results are those of separate buffers, in a call and in a drained
queue (where the batch after it reuses the copy's scratch)."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import ktype, log, new_pair, to_dev, to_host

pytestmark = pytest.mark.gpu


def _store(kb, seed):
    rng = np.random.default_rng(seed)
    s, o = new_pair(kb, cap=64, max_batch=1 << 18)
    k = w.KeySpace(kb, seed).build(60000)
    v = w.values_for(k, 2, kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    return s, o, k, rng


def _queries(rng, k, n, kb):
    return (k[rng.integers(0, k.size, n)] + rng.integers(0, 2, n).astype(ktype(kb))).astype(ktype(kb))


# offsets of an output in elements from the keys: in place, one lane, one wave,
# one workgroup, half the batch, before the keys
@pytest.mark.parametrize("kb,n", [(32, 200003), (64, 70001), (32, 300), (64, 1)])
@pytest.mark.parametrize("how", ["call", "drain"])
def test_point_reads_over_their_keys(kb, n, how):
    import torch
    s, o, k, rng = _store(kb, 5)
    dt = torch.int32 if kb == 32 else torch.int64
    ins = w.KeySpace(kb, 77).build(3000)
    iv = w.values_for(ins, 3, kb)
    for op in ("lookup", "successor", "predecessor"):
        for off in sorted({0, 1, 64, 256, -1, -64, n // 2, -(n // 2), n}):
            q = _queries(rng, k, n, kb)
            buf = torch.zeros(3 * n + 1024, dtype=dt, device="cuda")
            at = n + 256
            keys = buf[at: at + n]
            keys.copy_(to_dev(q))
            over = buf[at + off: at + off + n] if abs(off) <= n + 256 else None
            other = torch.zeros(n, dtype=dt, device="cuda")
            log(f"{how} {op} kb={kb} n={n} offset={off}")
            if op == "lookup":
                b = dict(op=op, keys=keys, out_v=over)
                want = [(over, o.lookup(q))]
            else:
                # the key output over the keys, then the value output over them
                wk, wv = o.successor(q) if op == "successor" else o.predecessor(q)
                if off % 2:
                    b = dict(op=op, keys=keys, out_k=over, out_v=other)
                    want = [(over, wk), (other, wv)]
                else:
                    b = dict(op=op, keys=keys, out_k=other, out_v=over)
                    want = [(other, wk), (over, wv)]
            if how == "call":
                getattr(s, op)(keys, *([b["out_v"]] if op == "lookup" else [b["out_k"], b["out_v"]]))
            else:
                s.drain([b, dict(op="insert", keys=to_dev(ins), aux=to_dev(iv)),
                         dict(op="delete", keys=to_dev(ins))])
            for t, x in want:
                assert np.array_equal(to_host(t, kb), x), f"{op} at offset {off}"
    assert s.status() == 0
    s.close()


@pytest.mark.parametrize("kb,n,maxpq", [(32, 60001, 4), (64, 30000, 3), (32, 70, 90), (64, 5000, 1)])
@pytest.mark.parametrize("how", ["call", "drain"])
def test_ranges_over_their_bounds(kb, n, maxpq, how):
    import torch
    s, o, k, rng = _store(kb, 6)
    dt = torch.int32 if kb == 32 else torch.int64
    order = np.sort(k)
    first = rng.integers(0, k.size - 200, n)
    lo, hi = order[first], order[first + rng.integers(0, 3 * maxpq // 2 + 2, n)]
    wc, wk, wv = o.range(lo, hi, maxpq)
    dhi = to_dev(hi)
    for which in ("out_k", "out_v", "counts"):
        size = n * maxpq
        buf = torch.zeros(size + 2 * n + 64, dtype=dt, device="cuda")
        at = size // 2 if which != "counts" else 33
        keys = buf[at: at + n]
        keys.copy_(to_dev(lo))
        outs = {x: torch.zeros(size, dtype=dt, device="cuda") for x in ("out_k", "out_v")}
        outs["counts"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        outs[which] = buf[:size] if which != "counts" else buf.view(torch.int32)[17: 17 + n]
        log(f"{how} ranges kb={kb} n={n} maxpq={maxpq} over={which}")
        if how == "call":
            s.range(keys, dhi, maxpq, counts=outs["counts"], out_k=outs["out_k"], out_v=outs["out_v"])
        else:
            s.drain([dict(op="range", keys=keys, aux=dhi, max_per_query=maxpq, **outs),
                     dict(op="delete", keys=to_dev(w.KeySpace(kb, 78).build(2000)))])
        c = outs["counts"].cpu().numpy().view(np.uint32)
        assert np.array_equal(c, wc)
        got = np.minimum(wc, maxpq)
        live = np.arange(maxpq)[None, :] < got[:, None]
        for t, x in ((outs["out_k"], wk), (outs["out_v"], wv)):
            a = to_host(t.contiguous(), kb).reshape(n, maxpq)
            assert np.array_equal(a[live], x.reshape(n, maxpq)[live])
    assert s.status() == 0
    s.close()


@pytest.mark.parametrize("kb", [32, 64])
def test_overlap_anywhere_in_a_long_queue(kb):
    import torch
    s, o, k, rng = _store(kb, 7)
    dt = torch.int32 if kb == 32 else torch.int64
    n = 3001
    queue, want = [], []
    for i in range(131):
        q = _queries(rng, k, n, kb)
        buf = torch.zeros(2 * n, dtype=dt, device="cuda")
        keys = buf[:n]
        keys.copy_(to_dev(q))
        off = 64 if i in (0, 5, 63, 64, 66, 127, 128, 130) else n
        queue.append(dict(op="lookup", keys=keys, out_v=buf[off: off + n]))
        want.append(o.lookup(q))
    log(f"drain of {len(queue)} lookups, kb={kb}")
    s.drain(queue)
    for i, (b, x) in enumerate(zip(queue, want)):
        assert np.array_equal(to_host(b["out_v"], kb), x), f"batch {i}"
    assert s.status() == 0
    s.close()
