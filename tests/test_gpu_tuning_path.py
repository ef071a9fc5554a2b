"""Which path a race check takes under a launch shape, seen in the stage times
of a profiling context, and that the autotuner's time is that of the calls
which follow it.  Results equal the oracle's on either path."""
import time

import numpy as np
import pytest

import oracle
import tracegen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def to_dev(recs):
    return torch.from_numpy(np.ascontiguousarray(recs).view(np.uint8).reshape(-1, 16)).to("cuda:0")


@pytest.mark.parametrize("blocks", [1, 16, 128])
@pytest.mark.parametrize("warp", [False, True])
def test_a_shape_asks_for_the_sort(blocks, warp):
    """A shape with a field set sorts; the default shape, set, counts by group
    (also below 2^20 records, which a profiling context sorts without one)."""
    import paper_1905_01833_amd as pkg

    recs, _ = tracegen.c1(n_blocks=blocks, inject_rate=1e-3, seed=blocks)
    side = (np.arange(len(recs)) % 5).astype(np.uint32)
    want = oracle.closed_form_warp(recs, side, None, 256) if warp else oracle.closed_form(recs, None, 256)
    dev, dside = to_dev(recs), torch.from_numpy(side.view(np.int32)).to("cuda:0")
    cls = pkg.sim_size_class(len(recs))
    c = pkg.Context(0, profile=True)
    try:
        for shape, sorts in (({"digit_bits": 8}, True), ({}, False), ({"group_shift_bias": -1}, True), (None, len(recs) < 1 << 20)):
            c.set_tuning(cls, shape)
            for rep in range(2):
                print(f"[gpu] {len(recs)} records, shape {shape}, warp-aware {warp}, call {rep}", flush=True)
                got = c.check_traces_warp_device(dev, dside, None, 256) if warp else c.check_traces_device(dev, None, 256)
                t = c.stage_times()
                assert (t["keygen"][1] > 0, t["filter_count"][1] > 0) == (sorts, not sorts), (shape, t)
                for a, b in zip(got, want):
                    assert a.tobytes() == b.tobytes(), shape
        c.set_tuning(cls + 1, {"digit_bits": 8})  # another class's shape says nothing about this one
        c.set_tuning(cls, {})
        (c.check_traces_warp_device(dev, dside, None, 256) if warp else c.check_traces_device(dev, None, 256))
        assert c.stage_times()["keygen"][1] == 0
    finally:
        c.close()


def test_autotune_times_the_calls_that_follow():
    """The stored shape's time is that of the calls that use it (noise and the
    least-of-few on both sides: within a factor of 1.7)."""
    import paper_1905_01833_amd as pkg

    recs, _ = tracegen.c1(n_blocks=1024, inject_rate=1e-4, seed=3)
    dev = to_dev(recs)
    want, wsum = oracle.closed_form_par(recs, tpb=256)
    c = pkg.Context(0)
    try:
        print("[gpu] autotune 2^24 records", flush=True)
        best = c.autotune(dev, None, 256, reps=5)
        took = []
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            got, gsum = c.check_traces_device(dev, None, 256)
            took.append((time.perf_counter() - t) * 1e3)
            assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes()
        print(f"[gpu] tuned {best['ms']:.3f} ms, calls {min(took):.3f} ms", flush=True)
        assert best["ms"] / 1.7 < min(took) < best["ms"] * 1.7
    finally:
        c.close()
