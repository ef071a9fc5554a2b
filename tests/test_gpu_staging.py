"""Staging overflow over more tiles than the GPU holds workgroups: tiles that
start after another tile's overflow must still report their counts."""
import numpy as np
import pytest

import tracegen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1 << 23, (1 << 23) + 4097])
def test_every_location_races_in_many_tiles(n):
    """Record pairs (2 i, 2 i + 1): two threads of one block write word i, so
    every location holds one racing pair (a last single record holds none)."""
    import paper_1905_01833_amd as pkg

    r = np.zeros(n, dtype=tracegen.RECORD_DTYPE)
    i = np.arange(n)
    r["unit"] = i // 2
    r["tid"] = i % 2
    r["action"] = tracegen.WRITE
    print(f"[gpu] staging overflow: {n} records", flush=True)
    ctx = pkg.Context(0)
    races, summ = ctx.check_traces_device(torch.from_numpy(r.view(np.uint8).reshape(-1, 16)).to("cuda:0"), None, 256)
    ctx.close()
    assert len(races) == n // 2 and int(summ[0]["n_pairs"]) == n // 2 and int(summ[0]["n_records"]) == n
    assert (races["unit"] == np.arange(n // 2)).all()
    for k, v in (("trace", 0), ("space", 0), ("kinds", 1), ("block", 0xFFFFFFFF), ("pairs_ww", 1), ("pairs_rw", 0),
                 ("pairs_aw", 0), ("pairs_ar", 0), ("pairs_xblock", 0)):
        assert (races[k] == v).all(), k
