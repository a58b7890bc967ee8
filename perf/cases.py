"""Performance cases of the library: what a user of it runs, over its range.

A case is a dict of plain values.  ``prepare`` makes, on the device and from
the seed alone, what a program holds before the call (the packed genomes and
the plan, workspace or server it keeps); ``run`` is one pass through the
public entry points; ``work`` gives the bytes that pass cannot do without.

Genomes are drawn as the repository's synthetic workloads are: related
genomes from one random base, with SNPs, indels of 1-10 bases, planted repeat
families and, where a case asks for them, runs of N.  The generator is plain
torch on the device, in pieces, so that a state's inputs are quick to make.

Entry points by ``kind``:
  run     Plan.run on a resident input (as bench.py times it), the results
          copied from the plan's memory into the program's own
  batch   the same for a plan of many independent sets
  ws      Plan.run_ws on caller-owned memory (no allocation, no host wait)
  build   twopaco_build: host genomes in, host result out
  serve   Server: a burst of jobs submitted at once, every result waited for
In ``build`` and ``serve`` the program copies each result out of the
library's block, so their genomes differ little (few junctions).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1602_05856_amd as tp

PIECE = 1 << 24  # bases made at a time


# ---------------------------------------------------------------- the cases

def _case(name, kind, genomes, length, k, h, filter="blocked", bits=16.0, snp=0.01, **more):
    c = dict(name=name, kind=kind, genomes=genomes, length=length, k=k, h=h, filter=filter,
             bits=bits, snp=snp, spread=0.0, indel=snp / 10, repeats=0.05, n_runs=0, rounds=1,
             strand="both", sets=1, hi=0)
    c.update(more)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest call: 4 genomes of 100 kbp, k = 25, b = 2^24, h = 3 (the
        # smoke test's workload), standard filter -- launches and host waits
        _case("tiny_standard", "run", 4, 100_000, 25, 3, "standard", 41.0),
        # the same on caller-owned memory: a serving loop that allocates nothing
        _case("tiny_ws", "ws", 4, 100_000, 25, 3, bits=41.0),
        # one small request from host memory to a host result (an odd size)
        _case("build_small", "build", 3, 700_001, 25, 4, snp=0.001),
        # 62 bacterial genomes of 5 Mbp at b = 2^30: the default k
        _case("bacterial_k25", "run", 62, 5_000_000, 25, 4, bits=2.5, snp=0.005, spread=0.015,
              indel=0.002),
        # ... with the paper's standard filter
        _case("bacterial_k25_standard", "run", 62, 5_000_000, 25, 4, "standard", 2.5, 0.005,
              spread=0.015, indel=0.002),
        # ... two-word k-mers
        _case("bacterial_k63", "run", 62, 5_000_000, 63, 4, bits=2.5, snp=0.005, spread=0.015,
              indel=0.002),
        # ... four-word k-mers
        _case("bacterial_k100", "run", 62, 5_000_000, 100, 4, bits=2.5, snp=0.005, spread=0.015,
              indel=0.002),
        # ... in four rounds (Algorithm 3), for a quarter of the exact table
        _case("bacterial_rounds", "run", 16, 5_000_000, 25, 4, bits=3.3, snp=0.005,
              spread=0.015, indel=0.002, rounds=4),
        # a batch of independent sets of uneven size, 50 kbp to 20 Mbp each
        _case("batch_k31", "batch", 6, 50_000, 31, 4, sets=128, hi=20_000_000),
        # a serving burst: small requests (k = 25) and two larger ones (k = 31)
        _case("serve_burst", "serve", 4, 300_000, 25, 4, snp=0.001, sets=12, hi=10_000_000),
        # a large request of the serving mix: 1 Gbp, k = 63
        _case("assembly_k63", "run", 5, 200_000_003, 63, 4),
        # primate-like genomes with repeat families and N runs, 1.6 Gbp (three
        # such states fit one GPU; the benchmark's 24 Gbp fits once)
        _case("primate_k25", "run", 8, 200_000_000, 25, 5, bits=4.0, snp=0.005, spread=0.035,
              indel=0.002, repeats=0.3, n_runs=25),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "run", "ws", "batch", "build", "serve"])
    filt = rng.choice(["blocked", "blocked", "blocked", "standard"])
    k = rng.choice([rng.randrange(15, 28), rng.randrange(28, 32), rng.randrange(32, 64),
                    rng.randrange(64, 128)])
    h = rng.choice([3, 4, 4, 5])
    bits = rng.choice([2.5, 4.0, 16.0, 16.0])
    snp = round(math.exp(rng.uniform(math.log(0.002), math.log(0.03))), 4)
    genomes = rng.randrange(2, 24)
    if kind == "batch":
        return _case(None, kind, rng.randrange(2, 8), _log(rng, 20_000, 200_000), k, h, filt, bits,
                     snp, sets=rng.randrange(3, 100), hi=_log(rng, 400_000, 20_000_000))
    if kind == "serve":
        return _case(None, kind, rng.randrange(2, 6), _log(rng, 50_000, 400_000), k, h,
                     "blocked", 16.0, min(snp, 0.002), sets=12, hi=_log(rng, 400_000, 8_000_000))
    # the largest total a case may have, by what its states hold
    top = 8_000_000 if kind == "build" else 40_000_000 if kind == "ws" else \
        200_000_000 if filt == "standard" or k > 63 or bits < 16 else 1_000_000_000
    total = _log(rng, 60_000, top)
    if kind == "build":
        snp = min(snp, 0.002)
    if total > 20_000_000:
        k = max(k, 21)  # shorter k-mers meet by chance everywhere at this size
    return _case(None, kind, genomes, max(200, total // genomes | 1), k, h, filt, bits, snp,
                 spread=rng.choice([0.0, snp]), n_runs=rng.choice([0, 0, 3]),
                 repeats=rng.choice([0.0, 0.05, 0.2]),
                 strand=rng.choice(["both", "both", "both", "both", "single"]),
                 rounds=rng.choice([1, 1, 1, 1, 2, 3]) if kind == "run" else 1)


# --------------------------------------------------------------- the inputs

def _gen(seed, *keys):
    g = torch.Generator(device="cuda")
    x = 0x9E3779B9
    for v in (seed,) + keys:
        x = (x * 1_000_003 + int(v) + 1) & 0x7FFFFFFFFFFF
    g.manual_seed(x)
    return g


def _codes(g, n):
    return torch.randint(0, 4, (n,), dtype=torch.uint8, device="cuda", generator=g)


def _plant(g, base, length, copies, divergence):
    """Copies of one random family of `length` bases, each at an offset of its
    own (places never overlap, so the result depends on the seed alone)."""
    places = base.numel() // length
    copies = min(copies, places)
    if copies < 1:
        return
    fam = _codes(g, length)
    at = torch.randperm(places, device="cuda", generator=g)[:copies] * length
    step = max(1, PIECE // length)
    for i in range(0, copies, step):
        a = at[i:i + step]
        x = fam.repeat(a.numel(), 1)
        hit = torch.rand(x.shape, device="cuda", generator=g) < divergence
        x = torch.where(hit, (x + torch.randint(1, 4, x.shape, dtype=torch.uint8, device="cuda",
                                                generator=g)) & 3, x)
        base[(a[:, None] + torch.arange(length, device="cuda")[None, :]).reshape(-1)] = \
            x.reshape(-1)


def _mutate(g, x, snp, indel):
    """SNPs at rate `snp`; indel events at rate `indel`, half deletions and
    half insertions of random bases, 1-10 long."""
    n = x.numel()
    r = torch.rand(n, device="cuda", generator=g)
    other = torch.randint(1, 4, (n,), dtype=torch.uint8, device="cuda", generator=g)
    x = torch.where(r < snp, (x + other) & 3, x)
    if not indel:
        return x
    at = torch.nonzero(r > 1 - indel).reshape(-1)
    if not at.numel():
        return x
    size = torch.randint(1, 11, (at.numel(),), device="cuda", generator=g)
    ins = torch.rand(at.numel(), device="cuda", generator=g) < 0.5
    gone = torch.zeros(n + 16, dtype=torch.bool, device="cuda")
    for j in range(10):
        gone[at[~ins & (size > j)] + j] = True
    copies = torch.ones(n, dtype=torch.int32, device="cuda")
    copies[gone[:n]] = 0
    copies[at[ins]] += size[ins].to(torch.int32)
    y = torch.repeat_interleave(x, copies)
    end = torch.cumsum(copies, 0)[at[ins]]
    k = size[ins]
    if k.numel():
        first = torch.repeat_interleave(end - k, k)
        run = torch.arange(first.numel(), device="cuda") - torch.repeat_interleave(
            torch.cumsum(k, 0) - k, k)
        y[first + run] = _codes(g, first.numel())
    return y


def _pack(x):
    n = x.numel()
    if n % 4:
        x = torch.cat([x, x.new_zeros(4 - n % 4)])
    x = x.view(-1, 4)
    return x[:, 0] | x[:, 1] << 2 | x[:, 2] << 4 | x[:, 3] << 6


def _genome_set(c, seed, key, n_genomes, length):
    """[(packed device tensor, bases, N runs)] of one set."""
    g = _gen(seed, key)
    base = _codes(g, length)
    if c["repeats"]:
        for flen, share in ((300, 0.4), (2000, 0.2), (6000, 0.4)):
            copies = int(c["repeats"] * share * length / flen)
            _plant(g, base, flen, copies, 0.05 if c["repeats"] < 0.1 else 0.15)
    out = []
    for i in range(n_genomes):
        g = _gen(seed, key, i)
        snp = c["snp"] + c["spread"] * i / max(1, n_genomes - 1)
        parts = [_mutate(g, base[a:a + PIECE], snp, c["indel"]) for a in range(0, length, PIECE)]
        # every genome is cut, or filled up with random bases, to the same length;
        # pieces are packed as they come: each but the last ends on a whole byte
        short = length - sum(p.numel() for p in parts)
        if short > 0:
            parts.append(_codes(g, short))
        packed, rest, n = [], None, 0
        for j, p in enumerate(parts):
            p = p[:length - n]
            n += p.numel()
            p = p if rest is None else torch.cat([rest, p])
            cut = p.numel() if j + 1 == len(parts) else p.numel() // 4 * 4
            packed.append(_pack(p[:cut]))
            rest = p[cut:]
            parts[j] = None
        runs = np.zeros((0, 2), np.uint64)
        if c["n_runs"]:
            r = np.random.RandomState((seed * 7919 + key * 131 + i) % (1 << 31))
            step = n // c["n_runs"]
            size = r.randint(1, max(2, min(10_000, step // 2)), c["n_runs"])
            start = np.arange(c["n_runs"]) * step + r.randint(0, max(1, step // 4), c["n_runs"])
            runs = np.stack([start, size], 1).astype(np.uint64)
        out.append((torch.cat(packed), n, runs))
    return out


def _sizes(c):
    """(genomes, genome length) of every set: one, or spread over [genomes *
    length, hi] in total, the same for every seed."""
    if c["sets"] == 1:
        return [(c["genomes"], c["length"])]
    r = np.random.RandomState(c["sets"])
    lo, hi = math.log(c["genomes"] * c["length"]), math.log(max(c["hi"], c["genomes"] * c["length"]))
    out = []
    for s in range(c["sets"]):
        g = 2 + s % max(1, 2 * c["genomes"] - 3)
        if c["kind"] == "serve":  # most requests small, two of them large
            total = c["hi"] * 4 if s % 6 == 3 else math.exp(lo + (hi - lo) * 0.5 * r.rand())
        else:
            total = math.exp(lo + (hi - lo) * r.rand())
        out.append((g, max(200, int(total / g) | 1)))
    return out


def _bits(c, bases):
    """Filter size: the power of two at or above c["bits"] per base."""
    b = 64
    while b < c["bits"] * bases:
        b <<= 1
    return b


def _flags(c):
    return (tp.TP_FLAG_BLOCKED_FILTER if c["filter"] == "blocked" else 0) | \
        (tp.TP_FLAG_SINGLE_STRAND if c["strand"] == "single" else 0)


class _View:
    """A device array of the library, for torch.as_tensor (no copy)."""

    def __init__(self, ptr, shape, typestr):
        self.__cuda_array_interface__ = dict(data=(ptr, False), shape=shape, typestr=typestr,
                                             version=3, strides=None)


def _take(dst, ptr, n, typestr="<i8"):
    """The first n rows of dst from a device array of the library."""
    if n > dst.shape[0]:
        raise RuntimeError("more results than the program has room for: %d of %d" % (
            n, dst.shape[0]))
    if n:
        dst[:n].copy_(torch.as_tensor(_View(ptr, (n,) + tuple(dst.shape[1:]), typestr),
                                      device="cuda"))


def _share(c, g, k):
    """Expected junctions per position of g genomes: a k-mer that keeps the
    base's sequence is one when another genome that keeps it differs next to
    it (a first and a last k-mer per string besides)."""
    d = c["snp"] + c["spread"] / 2 + 5 * c["indel"] / 2
    keep = (1 - c["snp"] - c["spread"] / 2 - c["indel"]) ** k
    return keep * (1 - (1 - min(1.0, 2 * d * keep)) ** (g - 1))


def _room(c, sets):
    """Junctions a program makes room for: half as many again as expected,
    short k-mers (which meet by chance) as many as there are positions."""
    n = sum(g * n for g, n in sets)
    if c["k"] < 21 or n < 4_000_000:
        return n
    more = sum(g * n * _share(c, g, c["k"]) for g, n in sets) * 1.5 + n * (0.03 + c["repeats"])
    return int(min(n, more + 1000))


def _serve_k(c, s):
    return 31 if c["kind"] == "serve" and s % 6 == 3 and c["k"] < 28 else c["k"]


def _host_room(c, gs, k):
    """The program's own host arrays for one result."""
    room = _room(c, [gs])
    return [np.zeros(gs[0] + 1, np.uint64), np.zeros(room, np.uint64),
            np.zeros((room, 1 if k <= 31 else 2 if k <= 63 else 4), np.uint64),
            np.zeros(room, np.uint8), np.zeros((room, 3), np.uint64)]


def prepare(case, seed):
    c = case
    sets = [_genome_set(c, seed, s, g, n) for s, (g, n) in enumerate(_sizes(c))]
    flags = _flags(c)
    total = [g * n for g, n in _sizes(c)]
    if c["kind"] in ("build", "serve"):
        host = [[tp.Genome(packed=p.cpu().numpy(), n_bases=n, n_runs=r) for p, n, r in gs]
                for gs in sets]
        outs = [_host_room(c, gs, _serve_k(c, s)) for s, gs in enumerate(_sizes(c))]
        if c["kind"] == "build":
            return dict(case=c, genomes=host[0], b=_bits(c, total[0]), flags=flags, out=outs[0])
        server = tp.Server(hbm_budget=24 << 30, workers=2, max_batch=8,
                           batch_max_bases=2_500_000, express_workers=1)
        return dict(case=c, server=server, flags=flags, out=outs,
                    jobs=[(gs, _serve_k(c, s), _bits(c, t))
                          for s, (gs, t) in enumerate(zip(host, total))])
    none = np.zeros(0, np.uint8)  # the sequences are on the device already
    listed_sets = [([tp.Genome(packed=none, n_bases=n, n_runs=r) for _, n, r in gs], _bits(c, t))
                   for gs, t in zip(sets, total)]
    if c["kind"] == "batch":
        plan = tp.Plan.batch(listed_sets, c["k"], c["h"], flags)
    else:
        plan = tp.Plan(listed_sets[0][0], c["k"], listed_sets[0][1], c["h"], flags)
        if c["rounds"] > 1:
            plan.rounds = c["rounds"]
    d_in = torch.zeros(plan.input_bytes, dtype=torch.uint8, device="cuda")
    i = 0
    for gs in sets:
        for p, _, _ in gs:
            o = plan.genome_offset(i)
            d_in[o:o + p.numel()] = p
            i += 1
    state = dict(case=c, plan=plan, d_in=d_in, n=i, W=1 if c["k"] <= 31 else 2 if c["k"] <= 63 else 4)
    if c["kind"] == "ws":
        # bounds that always hold; zeros, so that the unused tail is defined
        plan.workspace_layout(1.0, 1.0)
        ws, out = plan.alloc_workspace()
        out.zero_()
        plan.prepare_workspace(ws)
        state.update(ws=ws, out=out, views=plan.ws_views(out))
    else:
        # the program's own memory for the results (rows past the last are zero)
        room = _room(c, _sizes(c))
        i64 = dict(dtype=torch.int64, device="cuda")
        state["out"] = {
            "joff": torch.zeros(i + 1, **i64), "pos": torch.zeros(room, **i64),
            "vertex": torch.zeros((room, state["W"]), **i64),
            "strand": torch.zeros(room, dtype=torch.uint8, device="cuda"),
            "edges": torch.zeros((room, 3), **i64),
            "candidates": torch.zeros(plan.bitmap_words, **i64)}
    del sets, gs, p
    if sum(total) > PIECE:
        torch.cuda.empty_cache()  # the plan allocates its own device memory
    return state


# ---------------------------------------------------------------- one pass

def _host(out, r):
    """A host result's arrays into the program's own (an edge is three 64-bit
    words); the result block goes back to the library."""
    for dst, src in zip(out, (r.junction_offset, r.junction_pos, r.vertex, r.strand,
                              r.edges.view(np.uint64).reshape(-1, 3))):
        dst[:src.shape[0]] = src
    return out


def run(state):
    c = state["case"]
    if c["kind"] == "build":
        return _host(state["out"], tp.twopaco_build(state["genomes"], c["k"], state["b"], c["h"],
                                                    state["flags"]))
    if c["kind"] == "serve":
        srv = state["server"]
        ids = [srv.submit(gs, k, b, c["h"], state["flags"]) for gs, k, b in state["jobs"]]
        return [_host(o, srv.wait(i)[0]) for o, i in zip(state["out"], ids)]
    plan, out = state["plan"], state["out"]
    if c["kind"] == "ws":
        plan.run_ws(state["d_in"], state["ws"], out)
        return state["views"]
    plan.run(state["d_in"])
    o = plan.device_outputs()
    nj, ne = int(o["n_junctions"]), int(o["n_edges"])
    _take(out["joff"], o["junction_offset"], state["n"] + 1)
    _take(out["pos"], o["junction_pos"], nj)
    _take(out["vertex"], o["vertex"], nj)
    _take(out["strand"], o["strand"], nj, "|u1")
    _take(out["edges"], o["edges"], ne)
    _take(out["candidates"], o["candidates"], out["candidates"].numel())
    return out


def work(case):
    """The packed input read once and the results written once: the candidate
    bitmap, and per junction (as many as expected) its position, vertex,
    strand and edge."""
    c = case
    nbytes = 0.0
    for s, (g, n) in enumerate(_sizes(c)):
        k = _serve_k(c, s) if c["kind"] == "serve" else c["k"]
        W = 1 if k <= 31 else 2 if k <= 63 else 4
        nbytes += g * n * (0.25 + 0.125 + _share(c, g, k) * (8 + 8 * W + 1 + 24))
    return {"bytes": nbytes, "flops": 0}
