"""Barrier instances whose epoch runs begin and end anywhere: inside a word of
64 elements, across words, across tiles, at the ends of the trace."""
import numpy as np
import pytest

import oracle
from tracegen import RECORD_DTYPE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("length", [1, 2, 31, 63, 64, 65, 129, 4095, 4096, 4097, 9000])
def test_run_lengths(length, wide):
    """Words with epochs 0..4 (3 missing), runs of about `length` records, few
    writes and atomics, one or many threads."""
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(length)
    parts = []
    for word in range(max(2, min(400, 20000 // length))):
        threads = int(rng.choice([1, 2, 256]))
        for epoch in (0, 1, 2, 4):
            n = max(1, length + int(rng.integers(-1, 2)))
            r = np.zeros(n, dtype=RECORD_DTYPE)
            r["unit"] = word * (1 << 58 if wide and word < 30 else 1)
            r["tid"] = rng.integers(0, threads, n) + 256 * int(rng.integers(0, 2))
            r["epoch"] = epoch
            r["action"] = np.where(rng.random(n) < 0.5 / length, rng.integers(1, 3, n), 0)
            r["space"] = word & 1
            parts.append(r)
    recs = np.concatenate(parts)
    recs = recs[rng.permutation(len(recs))]
    off, tpb = np.array([0, len(recs)], dtype=np.uint64), np.array([256], dtype=np.uint32)
    print(f"[gpu] barrier runs of {length}: {len(recs)} records", flush=True)
    ctx = pkg.Context(0)
    races, summ, bar = ctx.check_sync_device(torch.from_numpy(recs.view(np.uint8).reshape(-1, 16)).to("cuda:0"), off, tpb)
    ctx.close()
    want, wsum = oracle.closed_form(recs, off, tpb)
    assert races.tobytes() == want.tobytes() and summ.tobytes() == wsum.tobytes()
    wbar = oracle.barriers(recs, off, tpb)
    assert len(wbar) and bar.tobytes() == wbar.tobytes()
