"""Cases that time the matching library through its public entry points.

Each case is one call (or, for the server, one burst of requests) as a user's
program makes it, on synthetic inputs of the shapes of ``synth/gen.py``, drawn
on the GPU so that they are quick to make:

  hyper   one hypergraph through ``match``: sizes uniform or Zipf(2.0), pins
          uniform or with Zipf(1.1) popularity, optionally one hub vertex in a
          quarter of the edges
  graph   one graph (two pins per edge) in the pair layout through ``match``:
          a random geometric graph or uniform endpoints
  batch   many small independent hypergraphs through ``match_batch``
  serve   a burst of host requests through ``Server``: submit all, poll until
          every bitmap is back

``stats`` says whether the caller asks for the per-round counts (the default
of ``match``) or only for the matching.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

import paper_2602_22976_amd as hgm

DEVICE = "cuda:0"


# ---------------------------------------------------------------------------
# The cases

def _hyper(n, m, smin, smax, weights, **kw):
    case = {"kind": "hyper", "n": n, "m": m, "smin": smin, "smax": smax, "sizes": "uniform",
            "pins": "uniform", "hub": False, "weights": weights, "variant": "auto",
            "vertex_side": True, "reseed": False, "stats": False}
    case.update(kw)
    return case


def _graph(shape, n, m, weights, **kw):
    case = {"kind": "graph", "shape": shape, "n": n, "m": m, "weights": weights,
            "vertex_side": True, "reseed": False, "stats": False}
    case.update(kw)
    return case


def listed():
    return [
        # The smallest call: a few hundred edges, where launches and the wait count.
        dict(_hyper(150, 311, 2, 8, 1000), name="tiny"),
        # The plain instance of the test suite, called with every default.
        dict(_hyper(10_000, 20_000, 2, 8, 1000, stats=True), name="plain-stats"),
        # An ordinary instance, odd sizes, only the matching wanted.
        dict(_hyper(60_013, 150_001, 2, 12, 1000), name="mid-uniform"),
        # The benchmark's instance as the benchmark calls it, per-round counts included.
        dict(_hyper(2_000_000, 5_000_000, 2, 64, 20, sizes="zipf", pins="zipf", stats=True),
             name="power-law-stats"),
        # The same shape for a program that only uses the matching.
        dict(_hyper(2_000_000, 5_000_000, 2, 64, 20, sizes="zipf", pins="zipf"),
             name="power-law"),
        # Cardinality matching with one vertex in a quarter of the edges.
        dict(_hyper(1_000_000, 4_000_000, 2, 16, 1, hub=True), name="hub-stress"),
        # Cardinality matching of a random geometric graph of 2^20 points.
        dict(_graph("rgg", 1 << 20, 6_850_001, 1), name="rgg"),
        # A weighted graph of ordinary size, with per-round counts.
        dict(_graph("uniform", 100_003, 399_989, 1_000_000, stats=True), name="graph-mid-stats"),
        # Priorities drawn afresh every round, only the edge side given.
        dict(_hyper(300_007, 700_001, 2, 64, 20, sizes="zipf", pins="zipf", reseed=True,
                    vertex_side=False), name="reseed-edge-side"),
        # The vertex-centric variant asked for by name.
        dict(_hyper(200_003, 499_979, 2, 12, 1000, variant="crew"), name="crew"),
        # The batched workload of the benchmark: 4,096 uneven small instances.
        {"name": "batch-4096", "kind": "batch", "count": 4096, "n_lo": 100, "n_hi": 50_000,
         "stats": False},
        # A burst at the request server, edge side only, eight workers.
        {"name": "serve-burst", "kind": "serve", "count": 64, "k_lo": 1_000, "k_hi": 1_000_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["hyper", "graph", "batch", "serve"], weights=[5, 2, 2, 1])[0]
    if kind == "hyper":
        kappa = _log_int(rng, 1_200, 36_000_000)
        zipf = rng.random() < 0.4
        smax = 64 if zipf else rng.choice([4, 8, 12, 16, 32])
        mean = 6.0 if zipf else (2 + smax) / 2
        m = max(64, int(kappa / mean) | 1)
        n = max(100, int(m * rng.uniform(0.3, 0.6)))
        weights = 20 if zipf else rng.choice([1, 1000, 1_000_000])
        variant = rng.choices(["auto", "crcw", "crew"], weights=[6, 1, 1])[0]
        side = variant == "crew" or rng.random() < 0.75
        hub = not zipf and rng.random() < 0.25
        reseed = rng.random() < 0.15
        stats = rng.random() < 0.4
        return _hyper(n, m, 2, smax, weights, sizes="zipf" if zipf else "uniform",
                      pins="zipf" if zipf else "uniform", hub=hub, variant=variant,
                      vertex_side=side, reseed=reseed, stats=stats)
    if kind == "graph":
        shape = rng.choice(["rgg", "uniform"])
        n = _log_int(rng, 2_000, 1_000_000)
        m = int(n * (0.4 * math.log(n) if shape == "rgg" else rng.uniform(2, 7))) | 1
        return _graph(shape, n, m, rng.choice([1, 1000, 1_000_000]),
                      vertex_side=rng.random() < 0.75, stats=rng.random() < 0.4)
    if kind == "batch":
        return {"kind": "batch", "count": _log_int(rng, 8, 2_000), "n_lo": 100,
                "n_hi": _log_int(rng, 1_000, 50_000), "stats": rng.random() < 0.3}
    return {"kind": "serve", "count": _log_int(rng, 12, 64), "k_lo": 1_000,
            "k_hi": _log_int(rng, 30_000, 1_000_000)}


# ---------------------------------------------------------------------------
# Inputs

def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _rand(gen, k):
    return torch.rand(k, dtype=torch.float64, device=DEVICE, generator=gen)


def _zipf_cdf(lo, hi, s):
    p = torch.arange(lo, hi + 1, dtype=torch.float64, device=DEVICE) ** -s
    c = torch.cumsum(p, 0)
    return c / c[-1]


def _offsets(sizes):
    off = torch.zeros(sizes.numel() + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(sizes, 0, out=off[1:])
    return off


def _distinct_pins(sizes, sample):
    """Pins without repeats inside an edge, ascending in each edge; returns
    (edge of each pin, pin).  ``sample(edges)`` draws one pin for each entry."""
    eid = torch.repeat_interleave(torch.arange(sizes.numel(), device=DEVICE), sizes)
    key = torch.sort((eid << 32) | sample(eid)).values
    del eid
    at = None                                  # positions still to be checked (None: all)
    sub = key
    while sub.numel():
        dup = torch.zeros(sub.numel(), dtype=torch.bool, device=DEVICE)
        dup[1:] = sub[1:] == sub[:-1]
        if not bool(dup.any()):
            break
        bad = torch.zeros(sizes.numel(), dtype=torch.bool, device=DEVICE)
        bad[sub[dup] >> 32] = True
        sel = bad[sub >> 32]
        at = torch.nonzero(sel).flatten() if at is None else at[sel]
        sub, dup = sub[sel], dup[sel]
        e = sub[dup] >> 32
        sub[dup] = (e << 32) | sample(e)
        sub = torch.sort(sub).values           # same edges in the same order
        key[at] = sub
    return key >> 32, key & 0xFFFFFFFF


def _weights(gen, m, weights):
    if weights == 1:
        return torch.ones(m, dtype=torch.int32, device=DEVICE)
    if weights == 20:                          # log-uniform in [1, 2^20]
        return torch.floor(torch.exp2(20.0 * _rand(gen, m))).clamp(1, 2 ** 20).to(torch.int32)
    return torch.randint(1, weights + 1, (m,), device=DEVICE, generator=gen).to(torch.int32)


def _vertex_side(n, eid, pins, edge_of=None):
    v_off = _offsets(torch.bincount(pins, minlength=n)).to(torch.int32)
    order = torch.sort((pins << 32) | eid).values & 0xFFFFFFFF
    return v_off, (order if edge_of is None else order - edge_of[order]).to(torch.int32)


def _hyper_arrays(case, seed):
    gen = _gen(seed)
    n, m = case["n"], case["m"]
    smax = min(case["smax"], n // 2)
    if case["sizes"] == "zipf":
        sizes = 2 + torch.searchsorted(_zipf_cdf(2, smax, 2.0), _rand(gen, m)).clamp(max=smax - 2)
    else:
        sizes = torch.randint(case["smin"], smax + 1, (m,), device=DEVICE, generator=gen)
    if case["pins"] == "zipf":
        cdf = _zipf_cdf(1, n, 1.1)
        perm = torch.randperm(n, device=DEVICE, generator=gen)

        def sample(edges):
            return perm[torch.searchsorted(cdf, _rand(gen, edges.numel())).clamp(max=n - 1)]
    else:
        def sample(edges):                     # vertex n - 1 is left for the hub
            return torch.randint(0, n - 1, (edges.numel(),), device=DEVICE, generator=gen)
    eid, pins = _distinct_pins(sizes, sample)
    off = _offsets(sizes)
    if case["hub"]:
        edges = torch.randperm(m, device=DEVICE, generator=gen)[:m // 4]
        pins[off[edges + 1] - 1] = n - 1       # the last pin: the order stays ascending
    return eid, off, pins, _weights(gen, m, case["weights"])


def _rgg_pairs(gen, n, m):
    """m pairs of points closer than 0.55 sqrt(ln n / n) in the unit square (a
    few percent fewer than there are), by a grid of cells of that size (own
    cell and four of the eight neighbours)."""
    r = 0.55 * math.sqrt(math.log(n) / n)
    side = max(1, int(1.0 / r))
    pts = torch.rand((n, 2), dtype=torch.float64, device=DEVICE, generator=gen)
    cxy = (pts * side).long().clamp(max=side - 1)
    cell, order = torch.sort(cxy[:, 0] * side + cxy[:, 1])
    start = torch.searchsorted(cell, torch.arange(side * side + 1, device=DEVICE))
    me = torch.arange(n, device=DEVICE)
    keys = []
    for dx, dy in ((0, 0), (1, -1), (1, 0), (1, 1), (0, 1)):
        x, y = cxy[order, 0] + dx, cxy[order, 1] + dy
        ok = (x >= 0) & (x < side) & (y >= 0) & (y < side)
        c = torch.where(ok, x * side + y, torch.zeros_like(x))
        lo, hi = start[c], start[c + 1]
        if dx == 0 and dy == 0:
            lo = torch.maximum(lo, me + 1)
        cnt = torch.where(ok, (hi - lo).clamp(min=0), torch.zeros_like(lo))
        first = lo - (torch.cumsum(cnt, 0) - cnt)
        src = torch.repeat_interleave(me, cnt)
        dst = first[src] + torch.arange(src.numel(), device=DEVICE)
        i, j = order[src], order[dst]
        near = ((pts[i] - pts[j]) ** 2).sum(1) < r * r
        i, j = i[near], j[near]
        keys.append(torch.minimum(i, j) * n + torch.maximum(i, j))
    key = torch.cat(keys)
    key = torch.sort(key[torch.randperm(key.numel(), device=DEVICE, generator=gen)[:m]]).values
    return torch.stack([key // n, key % n], 1)


def _graph_arrays(case, seed):
    gen = _gen(seed)
    n = case["n"]
    if case["shape"] == "rgg":
        pairs = _rgg_pairs(gen, n, case["m"])
    else:
        a = torch.randint(0, n, (case["m"],), device=DEVICE, generator=gen)
        b = (a + torch.randint(1, n, (case["m"],), device=DEVICE, generator=gen)) % n
        pairs = torch.stack([torch.minimum(a, b), torch.maximum(a, b)], 1)
    m = pairs.shape[0]
    eid = torch.repeat_interleave(torch.arange(m, device=DEVICE), 2)
    off = 2 * torch.arange(m + 1, device=DEVICE)
    return eid, off, pairs.reshape(-1).contiguous(), _weights(gen, m, case["weights"])


def _many_arrays(gen, ns, ms, smax, weights):
    """Instances of ns[i] vertices and ms[i] edges as their disjoint union:
    bases, instance of each edge, edge of each pin, sizes, global pins, weights."""
    vb, eb = _offsets(ns), _offsets(ms)
    inst = torch.repeat_interleave(torch.arange(ns.numel(), device=DEVICE), ms)
    sizes = torch.randint(2, smax + 1, (inst.numel(),), device=DEVICE, generator=gen)
    n_of = ns[inst]

    def sample(edges):
        return (_rand(gen, edges.numel()) * n_of[edges]).long()

    eid, pins = _distinct_pins(sizes, sample)
    return vb, eb, inst, eid, sizes, pins, _weights(gen, inst.numel(), weights)


def _log_sizes(count, lo, hi):
    """count sizes log-uniform in [lo, hi], the same for every seed."""
    return torch.exp(math.log(lo) + math.log(hi / lo) * _rand(_gen(1004), count)).round().long()


def _batch_sizes(case):
    ns = _log_sizes(case["count"], case["n_lo"], case["n_hi"])
    return ns, 2 * ns


def _serve_sizes(case):
    ms = _log_sizes(case["count"], case["k_lo"] / 17, case["k_hi"] / 17)
    return (ms // 2).clamp(min=64), ms


def _local_offsets(off, eb):
    """Offsets of each instance from 0, one extra entry per instance."""
    count = eb.numel() - 1
    idx = torch.arange(off.numel() - 1 + count, device=DEVICE)
    inst = torch.searchsorted(eb[1:] + torch.arange(1, count + 1, device=DEVICE), idx, right=True)
    return (off[idx - inst] - off[eb[inst]]).to(torch.int32)


def _priority_seed(seed):
    return 1 + seed % 1000


# ---------------------------------------------------------------------------
# What a program holds before the call

def prepare(case, seed):
    if case["kind"] == "batch":
        return _prepare_batch(case, seed)
    if case["kind"] == "serve":
        return _prepare_serve(case, seed)
    pairs = case["kind"] == "graph"
    eid, off, pins, w = (_graph_arrays if pairs else _hyper_arrays)(case, seed)
    none = torch.empty(0, dtype=torch.int32, device=DEVICE)
    v_off, v_edges = _vertex_side(case["n"], eid, pins) if case["vertex_side"] else (none, none)
    g = hgm.DeviceHypergraph(case["n"], w.numel(), off.to(torch.int32), pins.to(torch.int32),
                             v_off, v_edges, w)
    opts = hgm.make_opts("auto" if pairs else case["variant"], reseed=case["reseed"], pairs=pairs)
    return {"kind": case["kind"], "g": g, "seed": _priority_seed(seed), "opts": opts,
            "workspace": hgm.alloc_workspace(g, opts),
            "bits": torch.empty((g.m + 31) // 32, dtype=torch.int32, device=DEVICE),
            "stats": case["stats"]}


def _prepare_batch(case, seed):
    gen = _gen(seed)
    ns, ms = _batch_sizes(case)
    vb, eb, inst, eid, sizes, pins, w = _many_arrays(gen, ns, ms, 12, 1000)
    off = _offsets(sizes)
    wb = _offsets((ms + 31) // 32)
    v_off, v_edges = _vertex_side(int(vb[-1]), eid, pins + vb[inst[eid]], eb[inst])
    b = hgm.DeviceBatch(case["count"], int(vb[-1]), int(eb[-1]), int(off[-1]), int(wb[-1]), vb, eb,
                        off[eb], wb, _local_offsets(off, eb), pins.to(torch.int32),
                        _local_offsets(v_off.long(), vb), v_edges, w,
                        torch.arange(case["count"], dtype=torch.int32, device=DEVICE))
    opts = hgm.make_opts()
    return {"kind": "batch", "g": b, "opts": opts, "workspace": hgm.alloc_batch_workspace(b, opts),
            "bits": torch.empty(b.words_total, dtype=torch.int32, device=DEVICE),
            "stats": case["stats"]}


def _pinned(t):
    host = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    host.copy_(t)
    return host


def _prepare_serve(case, seed):
    gen = _gen(seed)
    ns, ms = _serve_sizes(case)
    vb, eb, inst, eid, sizes, pins, w = _many_arrays(gen, ns, ms, 32, 1_000_000)
    off = _offsets(sizes)
    e_off, pins, w = _pinned(_local_offsets(off, eb)), _pinned(pins.to(torch.int32)), _pinned(w)
    pb, eb, ns = off[eb].tolist(), eb.tolist(), ns.tolist()
    none = np.zeros(0, np.int32)
    requests = []
    for i in range(case["count"]):
        requests.append(types.SimpleNamespace(
            n=ns[i], m=eb[i + 1] - eb[i], e_off=e_off[eb[i] + i:eb[i + 1] + i + 1].numpy(),
            e_pins=pins[pb[i]:pb[i + 1]].numpy(), v_off=none, v_edges=none,
            w=w[eb[i]:eb[i + 1]].numpy().view(np.uint32)))
    return {"kind": "serve", "requests": requests, "hold": (e_off, pins, w),
            "server": hgm.Server(2 << 30, workers=8, edge_side_only=True)}


# ---------------------------------------------------------------------------
# One pass

def run(state):
    if state["kind"] == "serve":
        server, out = state["server"], {}
        ids = [server.submit(g, seed=i) for i, g in enumerate(state["requests"])]
        while len(out) < len(ids):
            for res in server.poll(timeout_s=1.0):
                if res["status"] != hgm.HGM_OK:
                    raise RuntimeError(hgm.hgm_strerror(res["status"]))
                out[res["id"]] = res["bits"]
        return [out[i] for i in ids]
    if state["kind"] == "batch":
        bits, stats = hgm.match_batch(state["g"], state["opts"], state["workspace"], state["bits"],
                                      want_stats=state["stats"])
    else:
        bits, stats = hgm.match(state["g"], state["seed"], state["opts"], state["workspace"],
                                state["bits"], want_stats=state["stats"])
    return {"bits": bits, **_totals(stats)} if stats is not None else {"bits": bits}


ROWS = 64                                      # more rounds than any of these inputs takes
PER_ROUND = ("live_edges", "live_pins", "matched_per_round", "matched_pins")


def _totals(stats):
    """The counts as a program's log keeps them: totals, one row per round."""
    rows = np.zeros((ROWS, len(PER_ROUND)), dtype=np.int64)
    for k, name in enumerate(PER_ROUND):
        rows[:stats["rounds"], k] = stats[name]
    return {"rounds": stats["rounds"], "matched": stats["matched"], "weight": stats["weight"],
            "per_round": rows}


# ---------------------------------------------------------------------------
# Least work: the edge side and the weights read once, the bitmap written once
# (the vertex side is the same incidences again, and the call works without it).

def work(case):
    if case["kind"] == "batch":
        n = (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
        m = 2 * n * case["count"]
        kappa = 7 * m
    elif case["kind"] == "serve":
        kappa = (case["k_hi"] - case["k_lo"]) / math.log(case["k_hi"] / case["k_lo"])
        kappa *= case["count"]
        m = kappa / 17
    elif case["kind"] == "graph":
        m = case["m"]
        kappa = 2 * m
    else:
        m = case["m"]
        if case["sizes"] == "zipf":
            p = [k ** -2.0 for k in range(2, case["smax"] + 1)]
            mean = sum(k * q for k, q in enumerate(p, 2)) / sum(p)
        else:
            mean = (case["smin"] + case["smax"]) / 2
        kappa = mean * m
    offsets = 0 if case["kind"] == "graph" else 4 * m
    return {"bytes": int(4 * kappa + offsets + 4 * m + m / 8), "flops": 0}


# ---------------------------------------------------------------------------
# The matching by plain 64-bit tensor operations: rounds of local maxima.

def _hash(seed, ids):
    """MurmurHash3_x86_32 of the four little-endian bytes of ids (int64 tensors)."""
    full = 0xFFFFFFFF

    def rotl(x, r):
        return ((x << r) | (x >> (32 - r))) & full

    k = (rotl((ids * 0xCC9E2D51) & full, 15) * 0x1B873593) & full
    h = (rotl(seed ^ k, 13) * 5 + 0xE6546B64) & full
    h = h ^ 4
    h = ((h ^ (h >> 16)) * 0x85EBCA6B) & full
    h = ((h ^ (h >> 13)) * 0xC2B2AE35) & full
    return h ^ (h >> 16)


def _rounds(n, eid, pins, sizes, w, seeds, ids, reseed):
    """Matched edges (bool) and the per-round counts."""
    m = w.numel()
    w = w.long()
    matched = torch.zeros(m, dtype=torch.bool, device=DEVICE)
    live = torch.arange(m, device=DEVICE)
    counts = {name: [] for name in PER_ROUND}
    r = 0
    while live.numel():
        s = _hash(seeds[live], torch.full_like(live, r)) if reseed else seeds[live]
        key = torch.zeros(m, dtype=torch.int64, device=DEVICE)
        key[live] = (w[live] << 32) | _hash(s, ids[live])
        best = torch.full((max(n, 1),), -1, dtype=torch.int64, device=DEVICE)
        best.scatter_reduce_(0, pins, key[eid], "amax")
        lose = torch.zeros(m, dtype=torch.bool, device=DEVICE)
        lose[eid[best[pins] != key[eid]]] = True
        won = live[~lose[live]]
        matched[won] = True
        done = torch.zeros(max(n, 1), dtype=torch.bool, device=DEVICE)
        done[pins[matched[eid]]] = True
        gone = torch.zeros(m, dtype=torch.bool, device=DEVICE)
        gone[eid[done[pins]]] = True
        gone[won] = True
        counts["live_edges"].append(live.numel())
        counts["live_pins"].append(int(sizes[live].sum()))
        counts["matched_per_round"].append(won.numel())
        counts["matched_pins"].append(int(sizes[won].sum()))
        live = live[~gone[live]]
        keep = ~gone[eid]
        eid, pins = eid[keep], pins[keep]
        r += 1
    return matched, {"rounds": r, "matched": int(matched.sum()), "weight": int(w[matched].sum()),
                     **counts}


def _bitmap(matched):
    pad = torch.zeros((matched.numel() + 31) // 32 * 32, dtype=torch.int64, device=DEVICE)
    pad[:matched.numel()] = matched
    words = (pad.view(-1, 32) << torch.arange(32, device=DEVICE)).sum(1)
    return torch.where(words >= 2 ** 31, words - 2 ** 32, words).to(torch.int32)


def exact(case, seed):
    if case["kind"] in ("hyper", "graph"):
        hyper = case["kind"] == "hyper"
        eid, off, pins, w = (_hyper_arrays if hyper else _graph_arrays)(case, seed)
        ids = torch.arange(w.numel(), device=DEVICE)
        seeds = torch.full_like(ids, _priority_seed(seed))
        matched, stats = _rounds(case["n"], eid, pins, off[1:] - off[:-1], w, seeds, ids,
                                 case["reseed"])
        return {"bits": _bitmap(matched), **(_totals(stats) if case["stats"] else {})}
    gen = _gen(seed)
    batch = case["kind"] == "batch"
    ns, ms = (_batch_sizes if batch else _serve_sizes)(case)
    vb, eb, inst, eid, sizes, pins, w = _many_arrays(gen, ns, ms, 12 if batch else 32,
                                                     1000 if batch else 1_000_000)
    ids = torch.arange(w.numel(), device=DEVICE) - eb[inst]
    matched, stats = _rounds(int(vb[-1]), eid, pins + vb[inst[eid]], sizes, w, inst, ids, False)
    bits = [_bitmap(m) for m in matched.split(ms.tolist())]
    if batch:
        return {"bits": torch.cat(bits), **(_totals(stats) if case["stats"] else {})}
    return [b.cpu().numpy().view(np.uint32) for b in bits]
