"""The longest traces that count by group and the first one past them: the sizes
at which the partition takes its most buckets, and both sides of the line to the
sort, against the oracle."""
import numpy as np
import pytest

import oracle
from tracegen import ATOMIC, READ, RECORD_DTYPE, WRITE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def long_trace(n, seed):
    """A block per 2^17 records, each with the same reads of a part of its own, a
    few thousand writes in all, some of which race, and one word that many read,
    a few threads write, and others read in every block."""
    rng = np.random.default_rng(seed)
    m = 1 << 17
    one = np.zeros(m, dtype=RECORD_DTYPE)
    one["tid"] = rng.integers(0, 256, m)
    one["unit"] = rng.integers(0, 1 << 13, m)
    one["epoch"] = rng.integers(0, 3, m)
    r = np.resize(one, n)
    for k in range(0, n, m):
        r["tid"][k:k + m] += np.uint32(256 * (k // m))
        r["unit"][k:k + m] += np.uint64((k // m) << 13)
    w = rng.integers(0, n, 5000)
    r["action"][w] = rng.choice([WRITE, ATOMIC], len(w))
    hot = rng.integers(0, n, n // 50)
    r["unit"][hot], r["action"][hot] = 1 << 40, READ
    r["action"][hot[:5]] = WRITE
    last = n - 1 - np.arange(40)  # the ragged end races too
    r["unit"][last], r["action"][last], r["tid"][last] = (1 << 41) + np.arange(40) // 2, WRITE, np.arange(40)
    return r


@pytest.mark.parametrize("n,counted", [((1 << 26) + 1, True), ((1 << 26) + 16384, True), ((1 << 27) - 5000, True),
                                       (1 << 27, True), ((1 << 27) + 1, False)])
def test_ends_of_the_grouped_range(n, counted):
    import paper_1905_01833_amd as pkg

    recs = long_trace(n, seed=n % 1000)
    print(f"[gpu] {n} records: oracle", flush=True)
    want, wsum = oracle.closed_form_par(recs, tpb=256)
    c = pkg.Context(0, profile=True)
    try:
        dev = torch.from_numpy(recs.view(np.uint8).reshape(-1, 16)).to("cuda:0")
        for rep in range(2):
            print(f"[gpu] {n} records, call {rep}", flush=True)
            got, gsum = c.check_traces_device(dev, None, 256)
            assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes(), rep
            t = c.stage_times()
            assert (t["filter_count"][1] > 0, t["keygen"][1] > 0) == (counted, not counted), t
    finally:
        c.close()
    assert len(want) > 1000 and int(want["pairs_rw"].max()) > n // 50
