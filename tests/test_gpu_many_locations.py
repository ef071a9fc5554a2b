"""Calls with many racing locations: the sort's entries copied in order, the
grouped count's sorted and merged, and the line between the two; against the
oracle, and their cost against the kernels or the path beside them."""
import numpy as np
import pytest

import oracle
from test_gpu_racing import HOT, compare, private
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


@pytest.mark.parametrize("n_traces", [2, 64, 65, 300])
@pytest.mark.parametrize("count", [2049, 60000, 200000])
def test_one_trace_with_many_among_many_traces(n_traces, count):
    """The entries of one long trace are sorted by all workgroups, whatever the
    number of traces: the call takes at most twice the sort's time."""
    import time

    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(n_traces + count)
    long = locations(1 << 22, rng, count)
    parts = [private(1000 + 37 * (k % 50), rng) for k in range(n_traces - 1)]
    parts.insert(n_traces // 2, long)
    recs = np.concatenate(parts)
    off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.uint64)
    tpb = np.full(n_traces, 256, dtype=np.uint32)
    want, wsum = oracle.closed_form_par(recs, off, tpb)
    assert len(want) == count
    dev = device(recs)
    best = {}
    c = pkg.Context(0)
    try:
        for shape in (None, {"scatter_threads": 512}):
            c.set_tuning(pkg.sim_size_class(len(recs)), shape)
            took = []
            for rep in range(4):
                print(f"[gpu] {count} locations in one of {n_traces} traces, shape {shape}, call {rep}", flush=True)
                torch.cuda.synchronize()
                t = time.perf_counter()
                got, gsum = c.check_traces_device(dev, off, tpb)
                took.append(time.perf_counter() - t)
                assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes()
            best[shape is None] = min(took)
    finally:
        c.close()
    print(f"[gpu] {best[True] * 1e6:.0f} us, sorted {best[False] * 1e6:.0f}", flush=True)
    assert best[True] < 2 * best[False], best


@pytest.mark.parametrize("count", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, 900000])
def test_line_between_merging_and_sorting(count):
    """As many entries of a trace as are merged, and more: the first call costs at
    most twice the sort."""
    rng = np.random.default_rng(count)
    n = 1 << 24
    want = compare(f"{count} locations of 2^24 records", locations(n, rng, count), private(n, rng), 2.0)
    assert len(want) == count


@pytest.mark.parametrize("n_traces", [65, 300])
@pytest.mark.parametrize("count", [255, 256, 257, 1000, 2047, 2048])
def test_a_chunk_of_entries_among_many_traces(n_traces, count):
    """Up to a chunk of entries in one trace of many: their order is not left to
    one workgroup; the call takes at most twice the sort's time."""
    import time

    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(n_traces + count)
    parts = [private(300 + 7 * (k % 50), rng) for k in range(n_traces - 1)]
    parts.insert(n_traces // 2, locations(1 << 17, rng, count))
    recs = np.concatenate(parts)
    off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.uint64)
    tpb = np.full(n_traces, 256, dtype=np.uint32)
    want, wsum = oracle.closed_form_par(recs, off, tpb)
    assert len(want) == count
    dev = device(recs)
    best = {}
    c = pkg.Context(0)
    try:
        for shape in (None, {"scatter_threads": 512}):
            c.set_tuning(pkg.sim_size_class(len(recs)), shape)
            took = []
            for rep in range(6):
                print(f"[gpu] {count} locations in one of {n_traces} short traces, shape {shape}, call {rep}", flush=True)
                torch.cuda.synchronize()
                t = time.perf_counter()
                got, gsum = c.check_traces_device(dev, off, tpb)
                took.append(time.perf_counter() - t)
                assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes()
            best[shape is None] = min(took)
    finally:
        c.close()
    print(f"[gpu] {best[True] * 1e6:.0f} us, sorted {best[False] * 1e6:.0f}", flush=True)
    assert best[True] < 2 * best[False], best
