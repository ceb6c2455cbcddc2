"""A reserved value anywhere in an insert batch rejects the batch, also in the middle of
a run of keys longer than a share of the slice search that falls into one bucket."""
import numpy as np
import pytest

from paper_2604_16725_amd import workloads as w
from tests.gpu_helpers import assert_same_contents, ktype, log, new_pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kb,rb,algo", [(32, 8, "tl_bulk"), (64, 8, "tl_bulk"), (32, 4, "tl_bulk"),
                                        (64, 8, "st_tl_mixed")])
@pytest.mark.parametrize("n", [12288, 12289, 40000])
@pytest.mark.parametrize("how", ["call", "drain"])
def test_reserved_value_inside_a_dense_run(kb, rb, algo, n, how):
    from oracle.oracle import Oracle
    from paper_2604_16725_amd.flix import Store
    s = Store(key_bits=kb, capacity=64, radix_bits=rb, max_batch=1 << 16, insert_algo=algo)
    o = Oracle(kb)
    base = w.KeySpace(kb, 41).build(4000)
    v = w.values_for(base, 5, kb)
    s.bulk_load(to_dev(base), to_dev(v))
    o.bulk_load(base, v)
    run = np.sort(base)[1234] + np.arange(1, n + 1).astype(ktype(kb))
    for at in (0, 1500, n // 2, n - 1):
        rv = w.values_for(run, 8, kb)
        rv[at] = ktype(kb)((1 << kb) - 1)
        log(f"{how} kb={kb} rb={rb} {algo} n={n} reserved at {at}")
        if how == "call":
            s.insert(to_dev(run), to_dev(rv), check=False)
        else:
            s.drain([dict(op="insert", keys=to_dev(run), aux=to_dev(rv))])
        assert s.status() == -1
        assert_same_contents(s, o, kb, f"reserved at {at}")
    s.insert(to_dev(run), to_dev(w.values_for(run, 9, kb)))
    o.insert(run, w.values_for(run, 9, kb))
    assert s.status() == 0
    assert_same_contents(s, o, kb, "the run without it")
    s.close()
