"""Range and predecessor batches of a drained queue that later batches depend on, or
overwrite: through the counts, the keys and the values of a range (which span
n * max_per_query slots) and a predecessor's keys.  The results are those of the
same batches issued one by one."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import ktype, log, new_pair, to_dev

pytestmark = pytest.mark.gpu


def _run_one_by_one(s, batches):
    for b in batches:
        if b["op"] == "range":
            s.range(b["keys"], b["aux"], b["max_per_query"], counts=b["counts"], out_k=b["out_k"],
                    out_v=b["out_v"])
        elif b["op"] == "lookup":
            s.lookup(b["keys"], b["out_v"])
        else:
            getattr(s, b["op"])(b["keys"], b["out_k"], b["out_v"])


@pytest.mark.parametrize("kb,n,maxpq", [(32, 300, 5), (64, 4000, 7), (32, 70000, 2), (64, 50, 300)])
def test_dependencies_through_ranges_and_predecessors(kb, n, maxpq):
    import torch
    rng = np.random.default_rng(kb + n)
    s, _ = new_pair(kb, cap=64, max_batch=1 << 17)
    k = w.KeySpace(kb, 3).build(60000)
    v = k[rng.permutation(k.size)]                 # values are stored keys
    s.bulk_load(to_dev(k), to_dev(v))
    order = np.sort(k)
    dt = torch.int32 if kb == 32 else torch.int64

    def queue():
        r = np.random.default_rng(n)
        bufs = dict(rk=torch.zeros(n * maxpq, dtype=dt, device="cuda"),
                    rv=torch.zeros(n * maxpq, dtype=dt, device="cuda"),
                    c=torch.zeros(2 * n, dtype=torch.int32, device="cuda"))
        for x in ("pk", "pv", "sk", "sv", "l0", "l1", "l2", "q"):
            bufs[x] = torch.zeros(n, dtype=dt, device="cuda")
        b, q = bufs, []
        keep = []
        for rep in range(4):
            first = r.integers(0, k.size - 400, n)
            lo = to_dev(order[first])
            hi = to_dev(order[first + r.integers(0, maxpq + 3, n)])
            keep += [lo, hi]
            last = b["rk"][n * maxpq - n:], b["rv"][n * maxpq - n:]
            q += [dict(op="range", keys=lo, aux=hi, max_per_query=maxpq, counts=b["c"][:n],
                       out_k=b["rk"], out_v=b["rv"]),
                  # keys that the range wrote, at the far end of its span
                  dict(op="lookup", keys=last[0], out_v=b["l0"]),
                  dict(op="predecessor", keys=last[1], out_k=b["pk"], out_v=b["pv"]),
                  # keys that the predecessor wrote; over keys that it read
                  dict(op="successor", keys=b["pv"], out_k=b["sk"], out_v=last[1]),
                  dict(op="lookup", keys=b["sk"], out_v=b["l1"])]
            if kb == 32:                           # the counts as keys, then over them
                q += [dict(op="lookup", keys=b["c"][:n], out_v=b["l2"]),
                      dict(op="predecessor", keys=b["l1"], out_k=b["c"][n // 2: n // 2 + n],
                           out_v=b["pv"])]
            # bounds that an earlier batch wrote
            q += [dict(op="lookup", keys=last[0], out_v=b["q"]),
                  dict(op="range", keys=b["q"], aux=b["sk"], max_per_query=1, counts=b["c"][:n],
                       out_k=b["l0"], out_v=b["l2"])]
        return bufs, q, keep

    want, qa, _ka = queue()
    _run_one_by_one(s, qa)
    torch.cuda.synchronize()
    got, qb, _kb = queue()
    log(f"drain of {len(qb)} dependent batches, kb={kb} n={n} maxpq={maxpq}")
    s.drain(qb)
    torch.cuda.synchronize()
    assert s.status() == 0
    for x in want:
        assert torch.equal(got[x], want[x]), x
    s.close()
