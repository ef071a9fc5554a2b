"""The work this library is used for, as cases that can be timed.

Every case is one call (or one burst of requests) through the Python binding
of the C ABI, on traces of the kind the library checks: blocks of threads that
make accesses between barriers, three quarters reads, shared windows of 48 KiB
per block, global reads Zipf(1.1) over a large region, private global writes,
and a small rate of injected races.  The sizes are those of the benchmark
workloads and of the tests, or lie between them.

A program keeps one context for its run and hands it trace after trace, so
the cases share one (a second option, launch-sequence replay, needs buffers
that stay, so a state with that option keeps a context of its own).
"""
import math

import numpy as np
import torch

import paper_1905_01833_amd as pkg

DEV = "cuda:0"
MAX_RECORDS = 1 << 28    # records of the largest single trace
BATCH_TRACES = 4096      # traces of the largest batch
CHUNK = 1 << 26          # records generated at once

_shared = {}


def _context():
    """The program's context (created once; grows its buffers on demand)."""
    if "ctx" not in _shared:
        _shared["ctx"] = pkg.Context(0)
    return _shared["ctx"]


def _server():
    """The program's server: the default two workers on one GPU, with buffers
    reserved for batches of 2^22 records."""
    if "srv" not in _shared:
        _shared["srv"] = pkg.Server(0, hbm_budget_bytes=32 << 30, max_batch_requests=512, reserve_records=1 << 22)
    return _shared["srv"]


# ------------------------------------------------------------------ the cases

def _case(name, op, **kw):
    c = {"name": name, "op": op, "traces": 1, "log2_min": 14.0, "log2_max": 14.0, "records": 0, "blocks": 0, "tpb": 256,
         "atomics": 0.0, "region_log2": 24, "inject": 1e-4, "graphs": False}
    c.update(kw)
    return c


def listed():
    return [
        # one small kernel under a debugger-like loop: a block of 256 threads, latency alone counts
        _case("one block, 1279 records", "check", records=1279, blocks=1, inject=2e-3),
        # the median serving request, its buffers refilled and its launches replayed
        _case("request 2^14, replayed", "check", records=1 << 14, blocks=4, graphs=True),
        # a kernel with blocks of 192 threads and a trace that ends anywhere
        _case("192 threads, 700001", "check", records=700_001, blocks=229, tpb=192),
        # one kernel launch of 1024 blocks, 64 accesses per thread
        _case("one trace 2^24", "check", records=1 << 24, blocks=1024),
        # the largest single trace: 8192 blocks of 512 threads, with atomics
        _case("one trace 2^28, atomics", "check", records=MAX_RECORDS, blocks=8192, tpb=512, atomics=0.05,
              region_log2=28, inject=1e-5),
        # many traces of uneven size in one call (the headline workload)
        _case("batch of 4096", "check", traces=BATCH_TRACES, log2_min=8.0, log2_max=20.0),
        # requests that arrive together at a server, lognormal sizes around 2^14
        _case("burst of 64 requests", "serve", traces=64),
        # one generation of the evolutionary input search: 50 candidates scored in one call
        _case("fitness of 50", "fitness", traces=50, log2_min=10.0, log2_max=17.0),
        # races and redundant barriers of one kernel launch
        _case("sync 2^22", "sync", records=1 << 22, blocks=256),
        # the warp-aware check of one kernel launch
        _case("warp 2^22", "warp", records=1 << 22, blocks=256),
        # barrier divergence of a batch of launches, blocks of 32 to 1024 threads
        _case("divergence of 512", "divergence", traces=512, log2_min=10.0, log2_max=17.0, tpb=0),
        # a trace that the simulator left in host memory
        _case("host 2^20", "host", records=1 << 20, blocks=64),
    ]


def draw(rng):
    """One more case of the ranges above."""
    op = rng.choice(["check", "check", "check", "batch", "batch", "serve", "fitness", "sync", "warp", "divergence",
                     "host"])
    tpb = rng.choice([32, 64, 96, 128, 192, 256, 256, 256, 384, 512, 768, 1024])

    def size(lo, hi):
        return int(2.0 ** rng.uniform(lo, hi)) | 1  # odd

    def one(kind, lo, hi, **kw):
        n = size(lo, hi)
        blocks = max(1, min(8192, int(n / tpb / 2.0 ** rng.uniform(3.0, 8.0))))
        return _case(None, kind, records=n, blocks=blocks, tpb=tpb, inject=10.0 ** rng.uniform(-5.0, -3.0),
                     atomics=rng.choice([0.0, 0.0, 0.05]), **kw)

    if op == "check":
        lo, hi = rng.choice([(8, 14), (14, 20), (20, 25), (25, 27.9)])
        c = one("check", lo, hi, graphs=hi <= 14 and rng.random() < 0.5)
    elif op == "batch":
        traces = int(2.0 ** rng.uniform(1, 12))
        hi = rng.uniform(10, min(20.0, 27.0 - math.log2(traces) + 3.0))
        c = _case(None, "check", traces=traces, log2_min=8.0, log2_max=hi, tpb=tpb, inject=10.0 ** rng.uniform(-5, -3))
    elif op == "serve":
        c = _case(None, "serve", traces=rng.randrange(8, 97))
    elif op == "fitness":
        c = _case(None, "fitness", traces=rng.randrange(2, 201), log2_min=8.0, log2_max=rng.uniform(10, 18), tpb=tpb)
    elif op == "divergence":
        c = _case(None, "divergence", traces=int(2.0 ** rng.uniform(0, 10)), log2_min=8.0,
                  log2_max=rng.uniform(10, 20), tpb=rng.choice([0, tpb]))
    elif op == "host":
        c = one("host", 10, 22)
    else:
        c = one(op, 12, 24)
    del c["name"]
    return c


# ------------------------------------------------------------------ the traces

def _shapes(case, seed):
    """Per trace: records, blocks, accesses per thread, threads per block."""
    rng = np.random.default_rng(seed ^ 0x5EED)
    t = case["traces"]
    if case["records"]:
        n = np.array([case["records"]], dtype=np.int64)
        blocks = np.array([case["blocks"]], dtype=np.int64)
    elif case["op"] == "serve":  # lognormal, median 2^14, clipped
        n = np.clip(np.round(np.exp(rng.normal(math.log(1 << 14), 1.5, t))), 256, 1 << 20).astype(np.int64)
        blocks = np.clip(-(-n // (256 * 64)), 1, 256)
    else:  # log-uniform: evenly spaced quantiles in random order, so that seeds differ little in total
        q = (rng.permutation(t) + rng.random(t)) / t
        n = np.round(2.0 ** (case["log2_min"] + (case["log2_max"] - case["log2_min"]) * q)).astype(np.int64)
        blocks = np.round(2.0 ** (8.0 * rng.random(t))).astype(np.int64)
    tpb = np.full(len(n), case["tpb"] or 256, dtype=np.int64)
    k = -(-n // (blocks * tpb))
    return n, blocks, k, tpb


def _generate(n, blocks, k, tpb, case, seed, out, side, m0, m):
    """Records of some whole traces into out (int64 [sum n, 2]) and, for the
    warp-aware check, their side words.

    Emission order: blocks in turn, statements round-robin over the block's
    threads.  Shared words of a block are written in one half of the window
    and read in the other half, the halves changing at every barrier, and a
    word is written by one thread per epoch, so nothing races but what is
    injected: m locations, the call's m0-th and following."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    total = int(n.sum())
    first = np.concatenate([[0], np.cumsum(n)])

    def per(v):  # a per-trace value for every record
        if len(n) == 1:
            return int(v[0])
        return torch.repeat_interleave(torch.from_numpy(np.asarray(v)).to(DEV), reps, output_size=total)

    reps = torch.from_numpy(n).to(DEV)
    i = torch.arange(total, device=DEV) - per(first[:-1])  # record within its trace
    p_tpb, p_k = per(tpb), per(k)
    t = i % p_tpb
    bj = i // p_tpb
    b, j = bj // p_k, bj % p_k
    del bj
    tid = b * p_tpb + t
    epoch = torch.clamp(j // 16, max=65535)
    u = torch.rand(total, generator=g, device=DEV)
    atomics = case["atomics"]
    action = (u >= 0.75).to(torch.int64)
    if atomics:
        action += (u >= 1.0 - atomics).to(torch.int64)
    write, atomic = action == 1, action == 2
    shared = (torch.rand(total, generator=g, device=DEV) < 0.5) & ~atomic
    # global: Zipf(1.1) ranks spread over the read region, private words after it, atomic bins after those
    region = 1 << case["region_log2"]
    v = torch.rand(total, generator=g, device=DEV, dtype=torch.float64)

    def zipf(v, size):  # inverse of the continuous law on [1, size + 1)
        top = 1.0 - (size + 1.0) ** -0.1
        return torch.clamp((1.0 - v * top) ** -10.0, max=float(size)).to(torch.int64) - 1

    unit = (zipf(v, region) * 0x9E3779B1) % region
    unit = torch.where(write, region + tid * p_k + j, unit)
    if atomics:
        bins = (zipf(v, 1 << 16) * 0x9E3779B1) % (1 << 16)
        unit = torch.where(atomic, region + per(blocks * tpb * k) + bins, unit)
    # shared: words q * tpb + owner, slots q of one parity written, of the other read
    slots = 12288 // p_tpb
    half = torch.clamp(slots // 2, min=1) if torch.is_tensor(slots) else max(1, slots // 2)
    pick = (v * 1048573.0).to(torch.int64)
    q = 2 * (pick % half) + ((epoch + action) & 1)
    owner = torch.where(write, (t + 37 * epoch) % p_tpb, (pick * 40503 + t) % p_tpb)
    unit = torch.where(shared, q * p_tpb + owner, unit)
    del u, v, q, owner, pick
    # injected races: m pairs of neighbouring threads of one block and epoch, each at a location of its own -- the
    # private word of one of them, a shared word, or a word of the read region (one of the hottest), which other threads
    # and other blocks may read as well
    if m:
        span = total // m
        at = torch.arange(m, device=DEV)
        x = at * span + 2 + torch.randint(0, span - 4, (m,), generator=g, device=DEV)

        def of(p):
            return p[x] if torch.is_tensor(p) else p

        x = torch.where(t[x] > 0, x, torch.where(i[x] + 1 < of(per(n)), x + 1, x - 1))
        y = x - 1
        kind, at = (at + m0) % 3, at + m0
        place = torch.where(kind == 0, region + tid[x] * of(p_k) + j[x],
                            torch.where(kind == 1, (at * 37 + 5) % 12288, (at * 0x9E3779B1) % region))
        unit[x], unit[y] = place, place
        shared[x], shared[y] = kind == 1, kind == 1
        # (in one warp and statement, only two writes race)
        action[x], action[y] = 1, (at % 2) * (kind != 2) if side is None else 1
    out[:, 0] = unit
    out[:, 1] = tid | (epoch << 32) | (action << 48) | (shared.to(torch.int64) << 56)
    if side is not None:  # eight statements; one warp access in twenty runs diverged
        warp = tid // 32 * 1031 + j
        div = ((warp * 0x9E3779B1) & 0xFFFFFFFF) % 20 == 0
        side[:] = ((j % 8) - (div.to(torch.int64) << 31)).to(torch.int32)


def prepare(case, seed):
    state = {"case": case}
    if case["op"] == "divergence":
        rng = np.random.default_rng(seed)
        n, _, _, _ = _shapes(case, seed)
        tpb = np.full(len(n), case["tpb"]) if case["tpb"] else rng.choice([32, 64, 96, 128, 192, 256, 512, 1024], len(n))
        blocks = np.maximum(1, n // tpb)
        off = np.concatenate([[0], np.cumsum(blocks * tpb)]).astype(np.uint64)
        g = torch.Generator(device=DEV).manual_seed(seed)
        total, n_blocks = int(off[-1]), int(blocks.sum())
        size = torch.from_numpy(np.repeat(tpb, blocks)).to(DEV)
        div = torch.zeros(n_blocks, dtype=torch.bool, device=DEV)
        div[torch.randperm(n_blocks, generator=g, device=DEV)[:_divergent(case)]] = True
        blk = torch.repeat_interleave(torch.arange(n_blocks, device=DEV), size, output_size=total)
        early = div[blk] & (torch.rand(total, generator=g, device=DEV) < 0.3)
        start = torch.cumsum(size, 0) - size  # a divergent block has a thread that leaves and one that stays
        early[start], early[start + 1] = div, False
        state["x"] = torch.where(early, torch.randint(0, 4, (total,), generator=g, device=DEV), 4).to(torch.int32)
        state["off"], state["tpb"], state["ctx"] = off, tpb.astype(np.uint32), _context()
        return state
    n, blocks, k, tpb = _shapes(case, seed)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.uint64)
    recs = torch.empty((int(off[-1]), 2), dtype=torch.int64, device=DEV)
    side = torch.empty(len(recs), dtype=torch.int32, device=DEV) if case["op"] == "warp" else None
    races, a = _races(case), 0
    while a < len(n):  # whole traces, about CHUNK records at a time
        z = a + 1
        while z < len(n) and int(off[z + 1] - off[a]) <= CHUNK:
            z += 1
        s = slice(int(off[a]), int(off[z]))
        m0, m1 = (races * int(off[q]) // int(off[-1]) for q in (a, z))
        _generate(n[a:z], blocks[a:z], k[a:z], tpb[a:z], case, seed * 1_000_003 + a, recs[s],
                  None if side is None else side[s], m0, m1 - m0)
        a = z
    torch.cuda.empty_cache()
    state["x"], state["off"], state["tpb"] = recs, off, tpb.astype(np.uint32)
    if case["op"] == "host":
        state["x"] = recs.cpu().numpy().view(pkg.RECORD_DTYPE).reshape(-1)
    if side is not None:
        state["side"] = side
    if case["op"] == "serve":
        state["srv"] = _server()
        state["x"] = [recs[int(off[i]):int(off[i + 1])] for i in range(len(n))]
    elif case["graphs"]:
        state["ctx"] = pkg.Context(0, graphs=True)
        state["stream"] = torch.cuda.Stream()
    else:
        state["ctx"] = _context()
    return state


# ------------------------------------------------------------------- one pass

def _words(a):
    """A structured result as whole 64-bit words (no copy)."""
    return a.view(np.int64)


def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "check":
        stream = s["stream"].cuda_stream if case["graphs"] else None
        races, summ = s["ctx"].check_traces_device(s["x"], s["off"], s["tpb"], stream=stream)
    elif op == "host":
        races, summ = s["ctx"].check_traces(s["x"], s["off"], s["tpb"])
    elif op == "warp":
        races, summ = s["ctx"].check_traces_warp_device(s["x"], s["side"], s["off"], s["tpb"])
    elif op == "sync":
        races, summ, bar = s["ctx"].check_sync_device(s["x"], s["off"], s["tpb"])
        return {"races": _words(races), "traces": _words(summ), "barriers": _words(bar)}
    elif op == "fitness":
        f = s["ctx"].eval_fitness_device(s["x"], s["off"], s["tpb"])
        return {"counts": _words(f).reshape(-1, 6)[:, :5], "fitness": f["fitness"]}
    elif op == "divergence":
        return {"blocks": _words(s["ctx"].check_divergence_device(s["x"], s["off"], s["tpb"]))}
    else:  # a burst: every request submitted, then every result collected
        srv = s["srv"]
        tickets = [srv.submit_device(x, None, int(t)) for x, t in zip(s["x"], s["tpb"])]
        got = [srv.wait(t) for t in tickets]
        return {"races": np.concatenate([_words(r) for r, _ in got]), "traces": np.concatenate([_words(m) for _, m in got])}
    return {"races": _words(races), "traces": _words(summ)}


def _records(case):
    """Records (threads, for divergence) of a case, without its seed."""
    if case["records"]:
        return case["records"]
    if case["op"] == "serve":
        return int(case["traces"] * (1 << 14) * math.exp(0.5 * 1.5 ** 2))
    lo, hi = case["log2_min"], case["log2_max"]
    mean = (2.0 ** hi - 2.0 ** lo) / ((hi - lo) * math.log(2.0)) if hi > lo else 2.0 ** lo
    return int(case["traces"] * mean)


def _races(case):
    """Racing locations of a call (a few even where the rate gives none)."""
    return max(8, int(case["inject"] * _records(case)))


def _divergent(case):
    """Divergent blocks of a call."""
    return max(1, int(0.01 * _records(case) / (case["tpb"] or 1024)))


def work(case):
    """Each input read once, each output written once (a location for every
    injected race, a summary or row for every trace)."""
    n = _records(case)
    if case["op"] == "divergence":
        return {"bytes": 4 * n + 24 * _divergent(case), "flops": 0}
    per_record = 20 if case["op"] == "warp" else 16
    out = 0 if case["op"] == "fitness" else 64 * _races(case)
    return {"bytes": per_record * n + out + 48 * case["traces"], "flops": 0}


def exact(case, seed):
    """The one output that is not a whole number: the fitness, from the sets
    of locations and (location, thread) pairs."""
    if case["op"] != "fitness":
        return None
    s = prepare(case, seed)
    off, tpb = s["off"].astype(np.int64), s["tpb"]
    out = np.ones(len(tpb), dtype=np.float64)
    for i in range(len(tpb)):
        r = s["x"][off[i]:off[i + 1]]
        word = r[:, 1]
        tid, shared = word & 0xFFFFFFFF, (word >> 56) & 1
        block = torch.where(shared.bool(), tid // int(tpb[i]), 0)
        loc = torch.stack([shared, block, r[:, 0]], dim=1)
        g = len(torch.unique(loc, dim=0))
        f = len(torch.unique(torch.cat([loc, tid[:, None]], dim=1), dim=0))
        out[i] = g / f
    return {"counts": None, "fitness": out}
