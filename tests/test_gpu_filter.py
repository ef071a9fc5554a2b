"""The grouped race count: entries and summaries equal the oracle's, byte for
byte, for every form of trace its hashes, tiles, buckets, rounds and fallbacks
can meet."""
import numpy as np
import pytest

import oracle
import tracegen
from tracegen import ATOMIC, READ, RECORD_DTYPE, WRITE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BATCH = 1 << 21
SINGLE = 1 << 23
GROUPED = 300


@pytest.fixture()
def ctx():
    import paper_1905_01833_amd as pkg

    c = pkg.Context(0)
    yield c
    c.close()


def device(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1, a.itemsize)).to("cuda:0")


def check(ctx, recs, off, tpb, name):
    print(f"[gpu] grouped count, {name}: {len(recs)} records, {len(off) - 1} traces", flush=True)
    off = np.asarray(off, dtype=np.uint64)
    tpb = np.broadcast_to(np.asarray(tpb, dtype=np.uint32), len(off) - 1)
    want, wsum = oracle.closed_form_par(recs, off, np.ascontiguousarray(tpb))
    for again in range(2):
        got, gsum = ctx.check_traces_device(device(recs), off, tpb)
        assert len(got) == len(want), (name, len(got), len(want))
        assert got.tobytes() == want.tobytes(), name
        assert gsum.tobytes() == wsum.tobytes(), name
    return want


def records(n, rng, blocks=64, tpb=256, units=1 << 22, p_write=0.1, p_atomic=0.0, p_shared=0.5, epochs=4):
    r = np.zeros(n, dtype=RECORD_DTYPE)
    r["tid"] = rng.integers(0, blocks * tpb, n)
    r["epoch"] = rng.integers(0, epochs, n)
    u = rng.random(n)
    r["action"] = np.where(u < p_write, WRITE, np.where(u < p_write + p_atomic, ATOMIC, READ))
    r["space"] = rng.random(n) < p_shared
    r["unit"] = np.where(r["space"] == 1, rng.integers(0, 12288, n), rng.integers(0, units, n))
    return r


def offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)


@pytest.mark.parametrize("tpb,blocks", [(1, 4096), (32, 300), (96, 100), (256, 64), (1000, 17), (1 << 20, 5)])
def test_block_sizes(ctx, tpb, blocks):
    """Shifted and divided block indices, up to thread ids near 2^32."""
    rng = np.random.default_rng(tpb)
    sizes = [BATCH // 16 + k for k in (-3, -2, -1, 0, 1, 2, 3, 5)] * 2
    recs = records(sum(sizes), rng, blocks, tpb)
    if tpb == 1000:  # the last block a 32-bit id reaches
        recs["tid"] += np.uint32(0xFFFFFFFF // 1000 - 20) * np.uint32(1000)
    assert len(check(ctx, recs, offsets(sizes), tpb, f"blocks of {tpb}")) > 100


@pytest.mark.parametrize("edge", [-1, 0, 1])
def test_tile_edges_and_empty_traces(ctx, edge):
    """Traces of whole filter tiles and one record more or less, of one
    record, and empty ones between them."""
    rng = np.random.default_rng(7 + edge)
    sizes = [0, 1, 16384 + edge, 0, 2, 32768 + edge, 255, 65536 + edge, 131072 + edge, 0, 131072, 16383] * 6 + [0]
    recs = records(sum(sizes), rng, units=1 << 18)
    assert len(recs) > BATCH
    check(ctx, recs, offsets(sizes), 256, f"edges {edge}")


@pytest.mark.parametrize("form", ["reads", "atomics", "private writes", "all race", "one word", "wide units", "far units",
                                  "half race"])
def test_contents(ctx, form):
    """No racing record, only racing records (the sorting path follows), and
    keys of more than 64 bits."""
    rng = np.random.default_rng(sum(form.encode()))
    sizes = [BATCH // 8] * 9
    n = sum(sizes)
    recs = records(n, rng)
    i = np.arange(n)
    if form == "reads":
        recs["action"] = READ
    elif form == "atomics":
        recs["action"] = ATOMIC
    elif form == "private writes":  # each thread reads and writes words of its own, again and again
        recs["action"] = i & 1
        recs["space"] = 0
        recs["unit"] = recs["tid"].astype(np.uint64) * 8 + i % 8
    elif form == "all race":
        recs["action"], recs["unit"], recs["tid"], recs["space"], recs["epoch"] = WRITE, i // 2, i % 2, 0, 0
    elif form == "one word":
        recs["unit"] = 5
    elif form == "wide units":  # spans near 2^64: two-word keys
        recs["unit"] = np.where(recs["space"] == 0, recs["unit"] * np.uint64(0x0000040000000001), recs["unit"])
    elif form == "far units":
        recs["unit"] += np.uint64(0x7F0000000000)
    else:
        recs["action"] = np.where(i % 8 == 0, WRITE, recs["action"])
        recs["unit"] = np.where(recs["space"] == 0, recs["unit"] % np.uint64(1 << 14), recs["unit"])
    want = check(ctx, recs, offsets(sizes), 256, form)
    assert (len(want) == 0) == (form in ("reads", "atomics", "private writes"))


@pytest.mark.parametrize("hot", ["read", "read and one write", "written", "atomic", "many"])
def test_hot_words(ctx, hot):
    """A word with a tenth of a long trace's records: buckets in several parts,
    more reads and writes than the lists hold."""
    rng = np.random.default_rng(len(hot))
    n = SINGLE + 12345
    recs = records(n, rng, blocks=512, p_write=0.02, p_shared=0.3)
    pick = rng.random(n) < 0.1
    k = 400 if hot == "many" else 1
    recs["unit"] = np.where(pick, (1 << 22) + rng.integers(0, k, n), recs["unit"])
    recs["space"] = np.where(pick, 0, recs["space"])
    act = {"read": READ, "read and one write": READ, "written": WRITE, "atomic": ATOMIC, "many": READ}[hot]
    recs["action"] = np.where(pick, act, recs["action"])
    if hot in ("read and one write", "many"):
        recs["action"][np.flatnonzero(pick)[:: 4000]] = WRITE
    check(ctx, recs, offsets([n]), 256, f"hot word, {hot}")


@pytest.mark.parametrize("n", [(1 << 25) - 1, (1 << 25) + 16384, 42454555])
def test_long_traces(ctx, n):
    """The most buckets of each partition kernel and the first sizes past it."""
    rng = np.random.default_rng(n)
    recs = np.tile(records(1 << 20, rng, blocks=1, p_write=0.0, units=1 << 14), (n >> 20) + 1)[:n]
    i = np.arange(n)
    recs["tid"] += (i >> 20).astype(np.uint32) * np.uint32(256)  # a block per copy
    recs["unit"] += (i >> 20).astype(np.uint64) << np.uint64(14)
    w = rng.integers(0, n, 3000)
    recs["action"][w] = WRITE
    assert len(check(ctx, recs, offsets([n]), 256, f"{n} records")) > 100


def test_generated_batch_and_shuffle(ctx):
    recs, off, tpb, _ = tracegen.batch(tracegen.c3_shapes(96, log2_max=17.0), inject_rate=1e-3)
    recs = np.concatenate([recs] * 4)
    off = np.concatenate([[0]] + [off[1:] + np.uint64(q) * off[-1] for q in range(4)]).astype(np.uint64)
    tpb = np.tile(tpb, 4)
    assert len(recs) > BATCH
    want = check(ctx, recs, off, tpb, "generated")
    rng = np.random.default_rng(3)
    for i in range(len(tpb)):
        s = slice(int(off[i]), int(off[i + 1]))
        recs[s] = recs[s][rng.permutation(s.stop - s.start)]
    assert check(ctx, recs, off, tpb, "shuffled").tobytes() == want.tobytes()


@pytest.mark.parametrize("sizes", [[1], [2, 0, 1], [17], [4095, 4096, 4097], [8191], [8192, 0, 8192], [8193, 5], [8192] * 40, [GROUPED], [GROUPED] * 301, [1] * 64 + [GROUPED] + [3] * 4000, [40000, 0, 17]])
def test_short_calls(ctx, sizes):
    """The smallest calls that count by group, of one trace and of many."""
    rng = np.random.default_rng(len(sizes))
    for p_write in (0.0, 0.3):
        recs = records(sum(sizes), rng, blocks=3, units=1 << 10, p_write=p_write, p_atomic=p_write / 8)
        check(ctx, recs, offsets(sizes), 256, f"{len(sizes)} short traces, writes {p_write}")


@pytest.mark.parametrize("writers", [15, 16, 17, 70, 1100])
@pytest.mark.parametrize("p_atomic", [0.0, 0.5])
def test_hot_word_of_many_writers(ctx, writers, p_atomic):
    """A word that many threads read and several write, some of them in one
    block and epoch: the buckets a later workgroup counts."""
    rng = np.random.default_rng(writers)
    n = 1 << 19
    recs = records(n, rng, blocks=40, p_write=0.02)
    at = rng.permutation(n)[: n // 8]
    recs["unit"][at], recs["space"][at], recs["action"][at] = 1 << 23, 0, READ
    recs["action"][at[:writers]] = np.where(rng.random(writers) < p_atomic, ATOMIC, WRITE)
    recs["tid"][at[: writers // 2]] = 5 * 256 + rng.integers(0, 8, writers // 2)
    want = check(ctx, recs, offsets([n]), 256, f"{writers} writers, {p_atomic} atomic")
    assert len(want) and want["pairs_rw"].max() > n // 16


@pytest.mark.parametrize("writes", [300, 500, 2000, 3000, 20000])
def test_rounds(ctx, writes):
    """More racing writes in one bucket than its table holds: rounds by slot,
    then (all of one word) the sorting path and the calls after it."""
    rng = np.random.default_rng(writes)
    for n, words in ((16384, writes), (16384, 1), (1 << 20, writes // 2)):
        recs = records(n, rng, p_write=0.0)
        k = min(writes, n // 2)
        at = rng.permutation(n)[: 2 * k]
        recs["unit"][at] = (1 << 23) + np.arange(2 * k) % words
        recs["space"][at] = 0
        recs["action"][at] = np.where(np.arange(2 * k) < k, WRITE, READ)
        check(ctx, recs, offsets([n]), 256, f"{writes} writes, {words} words")


@pytest.mark.parametrize("n_traces", [1, 2, 5])
@pytest.mark.parametrize("locations", [2047, 2049, 10000])
def test_many_entries(ctx, n_traces, locations):
    """Entries of a trace in one sorted chunk and in several, some of them
    found in several buckets (a shared word that races in every epoch)."""
    rng = np.random.default_rng(locations)
    n = 1 << 19
    parts = []
    for t in range(n_traces):
        r = records(n, rng, p_write=0.0, epochs=1)
        k = locations if t != 1 else 7
        at = rng.permutation(n)[: 8 * k].reshape(8, k)
        for q in range(8):
            word = np.arange(k) % 11000
            block = np.arange(k) // 11000
            r["unit"][at[q]] = (1 << 20) + word
            r["space"][at[q]] = np.arange(k) % 2
            r["tid"][at[q]] = block * 256 + q
            r["epoch"][at[q]] = q // 2
            r["action"][at[q]] = WRITE if q % 2 else READ
        parts.append(r)
    want = check(ctx, np.concatenate(parts), offsets([n] * n_traces), 256, f"{locations} locations")
    assert len(want) >= locations


def test_invalid_record_and_recovery(ctx):
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(11)
    sizes = [BATCH // 8] * 9
    recs = records(sum(sizes), rng)
    for field, bad in (("action", 3), ("space", 2)):
        r = recs.copy()
        at = sizes[0] * 4 + 77777
        r[field][at] = bad
        r[field][at + 100000] = bad
        with pytest.raises(pkg.SimError) as e:
            ctx.check_traces_device(device(r), offsets(sizes), 256)
        assert e.value.code == pkg.SIM_ERECORD and f"index {at} " in str(e.value)
    check(ctx, recs, offsets(sizes), 256, "after an error")


def test_warp_aware(ctx):
    rng = np.random.default_rng(12)
    sizes = [BATCH // 8 + 3] * 9
    recs = records(sum(sizes), rng, blocks=4, p_write=0.05)
    side = (rng.integers(0, 5, len(recs)) | np.where(rng.random(len(recs)) < 0.1, 1 << 31, 0)).astype(np.uint32)
    off, tpb = offsets(sizes), np.full(9, 256, dtype=np.uint32)
    want, wsum = oracle.closed_form_warp(recs, side, off, tpb)
    print(f"[gpu] grouped count, warp-aware: {len(recs)} records", flush=True)
    got, gsum = ctx.check_traces_warp_device(device(recs), torch.from_numpy(side.view(np.int32)).to("cuda:0"), off, tpb)
    assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes()


def test_server_batches():
    """Requests gathered from separate device tensors into one grouped call."""
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(13)
    reqs = [records(BATCH // 8 + 1001 * k, rng, blocks=8) for k in range(12)]
    want = [oracle.closed_form(r, np.array([0, len(r)], dtype=np.uint64), np.array([256], dtype=np.uint32)) for r in reqs]
    dev = [device(r) for r in reqs]
    torch.cuda.synchronize()
    print("[gpu] grouped count, server", flush=True)
    srv = pkg.Server(0, slots=1)
    try:
        for _ in range(2):
            tickets = [srv.submit_device(d, None, 256) for d in dev]
            for t, (w, s) in zip(tickets, want):
                got, gsum = srv.wait(t)
                assert got.tobytes() == w.tobytes() and gsum.tobytes() == s.tobytes()
    finally:
        srv.close()
