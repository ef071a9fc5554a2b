"""The grouped race count on the CPU (a model built on the product's own
hashes and pair test): its entries are the oracle's, byte for byte."""
import ctypes

import numpy as np
import pytest

import oracle
import tracegen
from test_host import _hostsim
from tracegen import ATOMIC, READ, RECORD_DTYPE, WRITE


def same_races(recs, off, tpb, side=None):
    """Compares with the oracle; returns its entries and the share of the
    records the model had to test one by one."""
    lib = _hostsim()
    lib.hs_group.restype = ctypes.c_int64
    lib.hs_group.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p,
                             ctypes.c_int, ctypes.c_void_p, ctypes.c_uint64, ctypes.POINTER(ctypes.c_uint64)]
    recs = np.ascontiguousarray(recs)
    off = np.asarray(off, dtype=np.uint64)
    tpb = np.ascontiguousarray(np.broadcast_to(np.asarray(tpb, dtype=np.uint32), len(off) - 1))
    want, _ = oracle.closed_form(recs, off, tpb) if side is None else oracle.closed_form_warp(recs, side, off, tpb)
    tested = ctypes.c_uint64(0)
    for backwards in (0, 1):
        out = np.zeros(len(recs) + 1, dtype=want.dtype)
        n = lib.hs_group(recs.ctypes.data, off.ctypes.data, len(off) - 1, tpb.ctypes.data,
                         None if side is None else side.ctypes.data, backwards, out.ctypes.data, len(out),
                         ctypes.byref(tested))
        assert n == len(want) and out[:n].tobytes() == want.tobytes()
    return want, tested.value / max(1, len(recs))


@pytest.mark.parametrize("warp", [False, True])
def test_tiny_traces(warp):
    """Dense collisions in few words, all action mixes and block sizes."""
    rng = np.random.default_rng(5 + warp)
    for _ in range(120):
        tpb = int(rng.integers(1, 90))
        parts = [tracegen.random_small(rng, int(rng.integers(0, 60)), units=int(rng.integers(1, 9)), tpb=tpb)
                 for _ in range(5)]
        off = np.concatenate([[0], np.cumsum([len(p) for p in parts])])
        n = int(off[-1])
        side = (rng.integers(0, 3, n) | np.where(rng.random(n) < 0.3, 1 << 31, 0)).astype(np.uint32) if warp else None
        same_races(np.concatenate(parts), off, tpb, side)


@pytest.mark.parametrize("tpb", [1, 32, 96, 256, 1 << 30])
@pytest.mark.parametrize("wide", [False, True])
def test_several_buckets(tpb, wide):
    """A trace of several buckets; units up to 2^64, threads up to 2^32."""
    rng = np.random.default_rng(tpb % 1000 + wide)
    n = 60000
    r = np.zeros(n, dtype=RECORD_DTYPE)
    r["tid"] = rng.integers(0, min(2 ** 32, 40 * tpb), n)
    r["epoch"] = rng.integers(0, 3, n) * (21845 if wide else 1)
    r["action"] = rng.choice([READ, READ, READ, WRITE, ATOMIC], n)
    r["space"] = rng.integers(0, 2, n)
    r["unit"] = rng.integers(0, 50000, n).astype(np.uint64) * np.uint64(2 ** 48 - 59 if wide else 1)
    want, _ = same_races(r, [0, n], tpb)
    assert len(want)


def test_few_records_are_tested_one_by_one():
    """Of a generated trace, without and with injected races: the records of
    the racing locations (a hot word's readers among them) and chance hits, a
    sixteenth of the records at most (an eighth of the slots hold a write,
    less than a quarter of the records write)."""
    for rate in (0.0, 1e-3):
        recs, _ = tracegen.c1(n_blocks=16, inject_rate=rate)
        want, tested = same_races(recs, [0, len(recs)], 256)
        words = {(int(e["space"]), int(e["block"]), int(e["unit"])) for e in want}
        block = np.where(recs["space"] == 1, recs["tid"] // 256, 0xFFFFFFFF)
        racing = sum((int(s), int(b), int(u)) in words for s, b, u in zip(recs["space"], block, recs["unit"]))
        assert tested <= racing / len(recs) + 1 / 16, (tested, racing)


@pytest.mark.parametrize("step", [1, 2, 32, 1024, 4096, 1 << 20, 1 << 32])
def test_strided_words_spread_over_buckets(step):
    """Regular strides fill the buckets evenly (an average bucket and six
    deviations)."""
    lib = _hostsim()
    n = 1 << 18
    r = np.zeros(n, dtype=RECORD_DTYPE)
    r["unit"] = np.arange(n, dtype=np.uint64) * np.uint64(step)
    lib.hs_filter_most.restype = ctypes.c_uint64
    lib.hs_filter_most.argtypes = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint32]
    for lgb in (4, 8):
        mean = n / (1 << lgb)
        assert lib.hs_filter_most(r.ctypes.data, n, lgb) < mean + 6 * mean ** 0.5, (step, lgb)


def test_guard_covers_every_sum_of_pairs():
    """The cross-block sum of a location holds its reads' pairs with all of the
    table and the table's own pairs: no call just below the guard wraps it."""
    lib = _hostsim()
    lib.hs_pair_sums.restype = ctypes.c_int
    lib.hs_pair_sums.argtypes = [ctypes.c_uint32]
    assert lib.hs_pair_sums(1024) == 0


@pytest.mark.parametrize("how", [2, 3, 4, 6, 8, 10, 12, 14])
@pytest.mark.parametrize("warp", [False, True])
def test_groups_rounds_and_thinning(how, warp):
    """Pairs from counts per group, in rounds by slot, and with atomics thinned
    out, alone and together: the same entries as pair by pair, and the oracle's."""
    lib = _hostsim()
    lib.hs_group.restype = ctypes.c_int64
    lib.hs_group.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p,
                             ctypes.c_int, ctypes.c_void_p, ctypes.c_uint64, ctypes.POINTER(ctypes.c_uint64)]
    rng = np.random.default_rng(how + 100 * warp)
    for n, units, blocks, tpb in ((40, 3, 2, 40), (300, 5, 3, 64), (2000, 300, 4, 33), (20000, 4000, 40, 96), (3000, 1, 2, 256)):
        r = np.zeros(n, dtype=RECORD_DTYPE)
        r["tid"] = rng.integers(0, blocks * tpb, n)
        r["epoch"] = rng.integers(0, 3, n)
        r["action"] = rng.choice([READ, READ, WRITE, ATOMIC], n)
        r["space"] = rng.integers(0, 2, n)
        r["unit"] = rng.integers(0, units, n)
        side = (rng.integers(0, 3, n) | np.where(rng.random(n) < 0.3, 1 << 31, 0)).astype(np.uint32) if warp else None
        off, tp = np.array([0, n], dtype=np.uint64), np.array([tpb], dtype=np.uint32)
        want, _ = oracle.closed_form(r, off, tp) if side is None else oracle.closed_form_warp(r, side, off, tp)
        out, tested = np.zeros(n + 1, dtype=want.dtype), ctypes.c_uint64(0)
        m = lib.hs_group(r.ctypes.data, off.ctypes.data, 1, tp.ctypes.data, None if side is None else side.ctypes.data, how,
                         out.ctypes.data, len(out), ctypes.byref(tested))
        assert m == len(want) and out[:m].tobytes() == want.tobytes(), (n, units)
