"""The conflict filter's decisions on the CPU (a model built on the product's
own hashes): the races of the records it keeps are the races of all records."""
import ctypes

import numpy as np
import pytest

import oracle
import tracegen
from test_host import _hostsim
from tracegen import ATOMIC, READ, RECORD_DTYPE, WRITE


def keep_of(recs, off, tpb, x_slots=2048, rounds=3):
    lib = _hostsim()
    lib.hs_filter.restype = None
    lib.hs_filter.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_int, ctypes.c_void_p]
    lib.hs_filter.argtypes[2] = ctypes.c_uint32
    keep = np.zeros(len(recs), dtype=np.uint8)
    lib.hs_filter(recs.ctypes.data, off.ctypes.data, len(off) - 1, tpb.ctypes.data, x_slots, rounds, keep.ctypes.data)
    return keep.astype(bool)


def same_races(recs, off, tpb, **kw):
    recs = np.ascontiguousarray(recs)
    off = np.asarray(off, dtype=np.uint64)
    tpb = np.ascontiguousarray(np.broadcast_to(np.asarray(tpb, dtype=np.uint32), len(off) - 1))
    keep = keep_of(recs, off, tpb, **kw)
    left = np.concatenate([[0], np.cumsum(keep)])[off.astype(np.int64)].astype(np.uint64)
    want, wsum = oracle.closed_form(recs, off, tpb)
    got, gsum = oracle.closed_form(np.ascontiguousarray(recs[keep]), left, tpb)
    assert got.tobytes() == want.tobytes()
    assert gsum["n_pairs"].tobytes() == wsum["n_pairs"].tobytes()
    return keep, want


@pytest.mark.parametrize("rounds", [0, 1, 3])
@pytest.mark.parametrize("x_slots", [8, 2048])
def test_tiny_traces(rounds, x_slots):
    """Dense collisions in few words, all action mixes and block sizes."""
    rng = np.random.default_rng(rounds * 100 + x_slots)
    for _ in range(60):
        tpb = int(rng.integers(1, 9))
        parts = [tracegen.random_small(rng, int(rng.integers(0, 60)), units=int(rng.integers(1, 9)), tpb=tpb)
                 for _ in range(5)]
        off = np.concatenate([[0], np.cumsum([len(p) for p in parts])])
        same_races(np.concatenate(parts), off, tpb, rounds=rounds, x_slots=x_slots)


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
    keep, want = same_races(r, [0, n], tpb)
    assert len(want) and keep.any()


def test_little_but_racing_locations_survives():
    """Of a generated trace, without and with injected races: the records of
    the racing locations (a hot word's readers among them) and chance hits."""
    for rate in (0.0, 1e-3):
        recs, _ = tracegen.c1(n_blocks=16, inject_rate=rate)
        keep, want = same_races(recs, [0, len(recs)], 256)
        words = {(int(e["space"]), int(e["block"]), int(e["unit"])) for e in want}
        block = np.where(recs["space"] == 1, recs["tid"] // 256, 0xFFFFFFFF)
        racing = sum((int(s), int(b), int(u)) in words for s, b, u in zip(recs["space"], block, recs["unit"]))
        assert keep.sum() <= racing + 0.002 * len(recs), (keep.sum(), racing)


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
