"""Calls whose short traces are sorted in LDS beside the other traces' passes:
all mixes of the sizes where a trace changes sides, call after call on streams
of the caller, with one-word and two-word keys."""
import numpy as np
import pytest

import oracle
import tracegen
from test_gpu_fitness import batch_of, wide_trace

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [[20000, 1], [16384, 16385], [4096, 4097, 40000], [100, 0, 70000, 16384, 16383], [30000, 30000],
                                   [30000] + [50] * 300])
@pytest.mark.parametrize("wide", [False, True])
def test_mixed_sizes(sizes, wide):
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(len(sizes) + wide)
    traces = [tracegen.random_small(rng, n, units=500, blocks=4, tpb=64, epochs=5) for n in sizes]
    if wide:
        traces.append(wide_trace(rng, 3000))
    recs, off = batch_of(traces)
    tpb = np.full(len(traces), 64, dtype=np.uint32)
    want_f = oracle.fitness(recs, off, tpb)
    want_r, want_s = oracle.closed_form(recs, off, tpb)
    ctx = pkg.Context(0)
    try:
        for k in range(4):
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                dev = torch.from_numpy(np.ascontiguousarray(recs).view(np.uint8).reshape(-1, 16)).to("cuda:0")
                print(f"[gpu] {sizes[:5]}, wide {wide}, call {k}", flush=True)
                got = ctx.eval_fitness_device(dev, off, tpb)
                races, sums = ctx.check_sync_device(dev, off, tpb)[:2]
            assert got.tobytes() == want_f.tobytes()
            assert races.tobytes() == want_r.tobytes() and sums.tobytes() == want_s.tobytes()
    finally:
        ctx.close()
