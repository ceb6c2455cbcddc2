"""Read batches of a drained queue run into one another; where one reads or
overwrites what another writes, the results are still those of running them
one by one.  Checked against the oracle applying the batches in order."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kb,n,depth", [(32, 1, 70), (32, 300, 200), (64, 5000, 66), (32, 70000, 9)])
def test_dependent_reads_in_one_drain(kb, n, depth):
    import torch
    from oracle.oracle import Oracle
    from paper_2604_16725_amd.flix import Store
    rng = np.random.default_rng(kb + n)
    # values are stored keys, so a lookup's answers are the next lookup's keys
    k = w.KeySpace(kb, 3).build(50000)
    v = k[rng.permutation(k.size)]
    s = Store(key_bits=kb, capacity=64, max_batch=1 << 17)
    o = Oracle(kb)
    s.bulk_load(to_dev(k), to_dev(v))
    o.bulk_load(k, v)
    dt = torch.int32 if kb == 32 else torch.int64
    buf = [torch.zeros(n, dtype=dt, device="cuda") for _ in range(2)]
    own = [torch.zeros(n, dtype=dt, device="cuda") for _ in range(depth)]
    tail = torch.zeros(n, dtype=dt, device="cuda")
    q0 = k[rng.integers(0, k.size, n)]
    q, cur, want_own = [], q0, []
    buf[0].copy_(to_dev(q0))
    ins = w.KeySpace(kb, 99).build(max(n, 100))
    iv = k[rng.integers(0, k.size, ins.size)]
    for i in range(depth):
        # independent read, then a read whose keys the previous one wrote and
        # whose output the one before that read (two buffers in turn)
        other = w.perm(rng.integers(0, 1 << 31, n, dtype=np.uint64), 7 + i, kb)
        q.append(dict(op="lookup", keys=to_dev(other), out_v=own[i]))
        q.append(dict(op="lookup", keys=buf[i % 2], out_v=buf[(i + 1) % 2]))
        if i == depth // 2:
            q.append(dict(op="insert", keys=to_dev(ins), aux=to_dev(iv)))
        want_own.append(o.lookup(other))
        cur = o.lookup(cur)
        if i == depth // 2:
            o.insert(ins, iv)
    # several batches into one output: the last one's answers stay
    for i in range(3):
        last = ins[rng.integers(0, ins.size, n)]
        q.append(dict(op="lookup", keys=to_dev(last), out_v=tail))
    ts = torch.full((len(q) + 1,), -1, dtype=torch.int64, device="cuda")
    log(f"drain of {len(q)} dependent batches, kb={kb} n={n}")
    for rep in range(2):   # the second run finds the first one's contents and buffers
        buf[0].copy_(to_dev(q0))
        s.drain(q, timestamps=ts)
        torch.cuda.synchronize()
        assert s.status() == 0
        t = ts.cpu().numpy()
        assert np.all(np.diff(t) >= 0) and t[0] > 0 and t[-1] > t[0]
        if rep == 0:
            for i in range(depth):
                assert np.array_equal(to_host(own[i], kb), want_own[i]), f"independent read {i}"
        if rep == 1:           # every read of the chain now follows the insert
            cur = q0
            for i in range(depth):
                cur = o.lookup(cur)
        assert np.array_equal(to_host(buf[depth % 2], kb), cur), f"chain of reads, run {rep}"
        assert np.array_equal(to_host(tail, kb), o.lookup(last)), f"shared output, run {rep}"
    s.close()
