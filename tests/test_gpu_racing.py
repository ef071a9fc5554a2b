"""Traces that race heavily: entries and summaries equal the oracle's, and a
call costs about what sorting its records costs, or less, whatever the words
that race look like (many writers and readers of a word, words written by
every thread, histograms, as many racing locations as there are words)."""
import time

import numpy as np
import pytest

import oracle
import tracegen
from tracegen import ATOMIC, READ, RECORD_DTYPE, WRITE

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HOT = 1 << 40


def private(n, rng, tpb=256):
    """A trace that does not race: a quarter of the records write words of
    their own, the others read a region that nobody writes."""
    r = np.zeros(n, dtype=RECORD_DTYPE)
    i = np.arange(n)
    k = -(-n // (max(1, n // (tpb * 64)) * tpb))
    r["tid"] = i // (tpb * k) * tpb + i % tpb
    w = rng.random(n) < 0.25
    r["action"] = np.where(w, WRITE, READ)
    r["unit"] = np.where(w, (1 << 24) + i, rng.integers(0, 1 << 24, n))
    return r


def writers(n, rng, count, readers):
    """`count` threads write one word, `readers` records read it."""
    r = private(n, rng)
    at = rng.permutation(n)[: count + readers]
    r["unit"][at] = HOT
    r["action"][at] = np.where(np.arange(len(at)) < count, WRITE, READ)
    return r


def call(ctx, dev, side=None):
    torch.cuda.synchronize()
    t = time.perf_counter()
    if side is None:
        got = ctx.check_traces_device(dev, None, 256)
    else:
        got = ctx.check_traces_warp_device(dev, side, None, 256)
    return got, time.perf_counter() - t


def compare(name, recs, clean, limit, warp=False):
    """The oracle's result, on a context's first call after one that did not
    race, and at most `limit` times what the call that sorts takes (the least
    of a few tries each)."""
    import paper_1905_01833_amd as pkg

    print(f"[gpu] racing, {name}: {len(recs)} records", flush=True)
    dev, cdev = (torch.from_numpy(np.ascontiguousarray(r).view(np.uint8).reshape(-1, 16)).to("cuda:0") for r in (recs, clean))
    side = dside = None
    if warp:
        side = (np.arange(len(recs)) % 7).astype(np.uint32)
        dside = torch.from_numpy(side.view(np.int32)).to("cuda:0")
        want, wsum = oracle.closed_form_warp(recs, side, None, 256)
    else:
        want, wsum = oracle.closed_form_par(recs, tpb=256)
    first, sort = [], []
    for _ in range(4):
        c = pkg.Context(0)
        try:
            call(c, cdev, dside)
            for k in range(3):
                (got, gsum), t = call(c, dev, dside)
                assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes(), (name, k)
                if k == 0:
                    first.append(t)
            c.set_tuning(pkg.sim_size_class(len(recs)), {"scatter_threads": 512})  # (the sort, in its default shape)
            for k in range(3):
                (got, gsum), t = call(c, dev, dside)
                assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes(), (name, "sorted", k)
                sort.append(t)
        finally:
            c.close()
    print(f"[gpu] {name}: {min(first) * 1e6:.0f} us, sorted {min(sort) * 1e6:.0f}, {len(want)} locations", flush=True)
    assert min(first) < limit * min(sort), (name, min(first), min(sort))
    return want


@pytest.mark.parametrize("warp", [False, True])
@pytest.mark.parametrize("log2", [10, 12, 13, 14, 16, 18, 20])
@pytest.mark.parametrize("count", [17, 100, 800])
def test_many_writers(log2, count, warp):
    """A word that many threads write and a fifth of the records read: in a
    trace counted from its records, one bucket, several, several parts."""
    rng = np.random.default_rng(log2)
    n = (1 << log2) - 3
    count = min(count, n // 8)
    want = compare(f"{count} writers of a word, 2^{log2}", writers(n, rng, count, n // 5), private(n, rng), 3.0, warp)
    assert len(want) >= 1 and int(want["pairs_rw"].max()) > n // 100


def flag(n, rng, share):
    """One word: a share of the records write it, as many read it."""
    m = int(n * share)
    return writers(n, rng, m, m)


def histogram(n, rng, bins):
    """Half of the records read and write bins, without atomics."""
    r = private(n, rng)
    at = rng.permutation(n)[: n // 2]
    r["unit"][at] = HOT + rng.integers(0, bins, len(at))
    r["action"][at] = np.arange(len(at)) % 2
    return r


def again(n, rng):
    """One thread writes a word again and again: no race."""
    r = private(n, rng)
    at = rng.permutation(n)[: n // 20]
    r["unit"][at], r["tid"][at], r["action"][at] = HOT, 7, WRITE
    return r


def counters(n, rng, reads):
    """A tenth of the records are atomics on four words, some reads among them."""
    r = private(n, rng)
    at = rng.permutation(n)[: n // 10]
    r["unit"][at], r["action"][at] = HOT + np.arange(len(at)) % 4, ATOMIC
    r["action"][at[:reads]] = READ
    return r


@pytest.mark.parametrize("log2", [12, 14, 16, 18, 20, 22])
@pytest.mark.parametrize("form", ["flag 5%", "flag 25%", "64 bins", "4096 bins", "one thread", "counters", "counters, read once",
                                  "counters, read often"])
def test_words_no_table_holds(log2, form):
    """Words with more writes than a table holds (and counters' atomics, which
    need none unless they meet a read): the call that finds out that it has to
    sort costs little more than the sort."""
    rng = np.random.default_rng(log2)
    n = (1 << log2) + 5
    make = {
        "flag 5%": lambda: flag(n, rng, 0.05), "flag 25%": lambda: flag(n, rng, 0.25),
        "64 bins": lambda: histogram(n, rng, 64), "4096 bins": lambda: histogram(n, rng, 4096),
        "one thread": lambda: again(n, rng), "counters": lambda: counters(n, rng, 0),
        "counters, read once": lambda: counters(n, rng, 1), "counters, read often": lambda: counters(n, rng, n // 100),
    }[form]
    want = compare(f"{form}, 2^{log2}", make(), private(n, rng), 3.0)
    assert (len(want) == 0) == (form in ("one thread", "counters"))


@pytest.mark.parametrize("n_blocks", [8, 32, 64, 256, 1024])
def test_hot_atomics_are_thinned_out(n_blocks):
    """Generated traces with one access in twenty atomic, most of them on a few
    hot words that nobody reads or writes: a bucket whose hot word shares its
    slot with a stranger's record is still counted, and the call does not sort."""
    import paper_1905_01833_amd as pkg

    c = pkg.Context(0, profile=True)
    try:
        for seed in range(4):
            recs, _ = tracegen.c2(n_blocks=n_blocks, inject_rate=0.0, seed=seed)
            want, wsum = oracle.closed_form_par(recs, tpb=512)
            print(f"[gpu] {len(recs)} records with atomics, seed {seed}", flush=True)
            c.set_tuning(pkg.sim_size_class(len(recs)), {})
            got, gsum = c.check_traces_device(torch.from_numpy(recs.view(np.uint8).reshape(-1, 16)).to("cuda:0"), None, 512)
            assert got.tobytes() == want.tobytes() and gsum.tobytes() == wsum.tobytes()
            t = c.stage_times()
            assert t["filter_count"][1] == 1 and t["keygen"][1] == 0, t
    finally:
        c.close()


@pytest.mark.parametrize("warp", [False, True])
def test_one_such_call_costs_the_others_nothing(warp):
    """After a call that had to sort, calls that need not are counted; a row of
    such calls is tried ever more rarely, and each kind of call by itself."""
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(5)
    n = 1 << 16
    racing, clean = flag(n, rng, 0.25), private(n, rng)
    side = np.zeros(n, dtype=np.uint32)
    dside = torch.from_numpy(side.view(np.int32)).to("cuda:0") if warp else None
    dev = [torch.from_numpy(r.view(np.uint8).reshape(-1, 16)).to("cuda:0") for r in (racing, clean)]
    want = [oracle.closed_form_warp(r, side, None, 256) if warp else oracle.closed_form(r, None, 256) for r in (racing, clean)]
    c = pkg.Context(0, profile=True)
    c.set_tuning(pkg.sim_size_class(n), {})
    try:
        def counted(k):
            print(f"[gpu] {'racing' if k == 0 else 'clean'} call, warp-aware {warp}", flush=True)
            got, _ = call(c, dev[k], dside)
            assert got[0].tobytes() == want[k][0].tobytes() and got[1].tobytes() == want[k][1].tobytes()
            t = c.stage_times()
            return t["filter_count"][1] > 0, t["keygen"][1] > 0

        assert counted(1) == (True, False)
        for _ in range(3):
            assert counted(0) == (True, True)  # tried, then sorted
            assert counted(1) == (True, False)
        tried = [counted(0)[0] for _ in range(40)]
        assert tried == [k in (0, 1, 3, 7, 15, 31) for k in range(40)]
        if warp:
            got, _ = c.check_traces_device(dev[1], None, 256)
            assert c.stage_times()["keygen"][1] == 0
    finally:
        c.close()


@pytest.mark.parametrize("warp", [False, True])
@pytest.mark.parametrize("n", [8190, 16384, (1 << 16) + 5, 1 << 19, (1 << 22) + 77])
@pytest.mark.parametrize("form", ["all write", "half atomic", "few words"])
def test_several_tables_of_candidates(form, n, warp):
    """Buckets whose candidates fill two to four tables: by later workgroups on
    the first call, by the first ones from then on, and as before again after a
    call that had none."""
    import paper_1905_01833_amd as pkg

    rng = np.random.default_rng(n)
    r = private(n, rng)
    if form == "all write":
        r["unit"], r["action"] = (1 << 24) + np.arange(n), WRITE
    elif form == "half atomic":
        at = rng.random(n) < 0.5
        r["unit"] = np.where(at, HOT + rng.integers(0, max(16, n // 128), n), r["unit"])
        r["action"] = np.where(at, ATOMIC, r["action"])
    else:  # words that a few threads of one block write and read, in every bucket
        at = rng.permutation(n)[: n // 2]
        r["unit"][at] = HOT + rng.integers(0, max(8, n // 8), len(at))
        r["tid"][at] = rng.integers(0, 3, len(at)) * 40
        r["action"][at] = rng.integers(0, 2, len(at))
    at = rng.permutation(n)[: 2 * (n // 500)]  # and pairs that race
    r["unit"][at], r["action"][at] = (1 << 41) + np.arange(len(at)) // 2, WRITE
    r["tid"][at] = np.arange(len(at)) % 2 * 100
    clean = private(n, rng)
    side = (np.arange(n) % 3).astype(np.uint32) if warp else None
    dside = torch.from_numpy(side.view(np.int32)).to("cuda:0") if warp else None
    sets = []
    for x in (r, clean):
        want = oracle.closed_form_warp(x, side, None, 256) if warp else oracle.closed_form_par(x, tpb=256)
        sets.append((torch.from_numpy(x.view(np.uint8).reshape(-1, 16)).to("cuda:0"), want))
    c = pkg.Context(0)
    try:
        for k, x in enumerate((0, 0, 0, 1, 0, 1, 1, 0)):
            print(f"[gpu] several tables, {form}, {n} records, warp-aware {warp}, call {k}", flush=True)
            (got, gsum), _ = call(c, sets[x][0], dside)
            assert got.tobytes() == sets[x][1][0].tobytes() and gsum.tobytes() == sets[x][1][1].tobytes(), (form, n, k)
    finally:
        c.close()
    assert len(sets[0][1][0]) >= n // 500


def read_often(n, rng, atomics, share):
    """`atomics` atomics on each of eight words that nobody writes, and a share
    of the records reads them."""
    r = private(n, rng)
    at = rng.permutation(n)[: int(n * share) + 8 * atomics]
    r["unit"][at], r["action"][at] = HOT + np.arange(len(at)) % 8, READ
    r["action"][at[: 8 * atomics]] = ATOMIC
    return r


@pytest.mark.parametrize("log2", [13, 16, 18, 20])
@pytest.mark.parametrize("atomics", [2, 16, 17, 100])
def test_reads_of_words_with_a_few_atomics(log2, atomics):
    """Many reads of words that a few atomics update and nobody writes: the sums
    of a word's pairs are kept together, not one for each of its atomics."""
    rng = np.random.default_rng(100 * log2 + atomics)
    n = (1 << log2) + 3
    want = compare(f"{atomics} atomics, 2^{log2}", read_often(n, rng, atomics, 0.4), private(n, rng), 3.0)
    assert len(want) == 8


@pytest.mark.parametrize("log2", [17, 19, 20, 22])
@pytest.mark.parametrize("others", [0, 7, 63])
def test_most_records_read_one_word(log2, others):
    """One word is read by half of a trace's records and others by the rest: the
    bucket of the first is split over workgroups wherever the others are, on every
    call (some calls left it whole)."""
    rng = np.random.default_rng(log2 + others)
    n = (1 << log2) + 7
    r = private(n, rng)
    at = rng.permutation(n)
    r["unit"], r["action"] = HOT + 1 + np.arange(n) % max(1, others), READ
    r["unit"][at[: n // 2]] = HOT
    r["action"][at[n // 2 - 10 : n // 2 + 40 * others]] = ATOMIC
    want = compare(f"half of 2^{log2} read a word, the others {others}", r, private(n, rng), 3.0)
    assert len(want) == 1 + others
