"""Calls with many racing locations: the sort's entries copied in order; against
the oracle, and their cost against the kernels beside them."""
import numpy as np
import pytest

import oracle
from test_gpu_racing import HOT, private
from tracegen import RECORD_DTYPE, WRITE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def locations(n, rng, count, base=None):
    """`count` words, each written by two threads."""
    r = private(n, rng) if base is None else base
    at = rng.permutation(n)[: 2 * count]
    r["unit"][at], r["action"][at] = HOT + np.arange(2 * count) % count, WRITE
    r["tid"][at] = np.arange(2 * count) // count + 2 * (np.arange(2 * count) % 7)
    return r


def device(r):
    return torch.from_numpy(np.ascontiguousarray(r).view(np.uint8).reshape(-1, 16)).to("cuda:0")


@pytest.mark.parametrize("log2,share", [(14, 12), (20, 12), (20, 64), (22, 12), (23, 12)])
def test_the_sorts_entries_are_copied_quickly(log2, share):
    """Copying the entries to their places takes at most twice what
    finding them in the sorted keys does, also where many of the words race
    (these lie spread among the others: the tiles' slices hold them, and the
    stages' times are those of the only scan)."""
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(log2 + share)
    n = (1 << log2) - 11
    recs = locations(n, rng, n // share)
    hot = recs["unit"] >= HOT
    recs["unit"][hot] = (recs["unit"][hot] - np.uint64(HOT)) * np.uint64(15485863) % np.uint64(1 << 24)
    want, wsum = oracle.closed_form_par(recs, tpb=256)
    dev = device(recs)
    c = pkg.Context(0, profile=True)
    try:
        c.set_tuning(pkg.sim_size_class(n), {"scatter_threads": 512})
        ratio = []
        for rep in range(4):
            print(f"[gpu] {len(want)} locations of {n} records, sorted, call {rep}", flush=True)
            got, gsum = c.check_traces_device(dev, None, 256)
            assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes()
            t = c.stage_times()
            ratio.append(t["scan_out"][0] / t["scan_tiles"][0])
        print(f"[gpu] copy {t['scan_out']} against scan {t['scan_tiles']}", flush=True)
        assert min(ratio) < 2, ratio
    finally:
        c.close()
