"""Performance cases of the library, over the range of calls a program makes.

A case is a dict of plain values; ``prepare`` makes its inputs on the GPU from a
seed, ``run`` takes one pass through the public entry points, ``work`` states
what a pass cannot do without, and ``exact`` gives a pass's answers from plain
numpy where that is quick.

Three kinds of pass:
  build   one text: ``Context.build``, then the tree read out (every level's
          marks and pointers into device tensors, the leaf bytes into pinned
          host memory) and freed.  With rank/select support the pass also
          answers one batch of rank and select queries.
  batch   many texts: ``Context.build_batch``, every tree read out and freed.
  query   ``Tree.access``, ``Tree.rank`` and ``Tree.select`` of one batch of m
          positions each against a resident tree.

Texts are repetitive ones: "dna" is a random ACGT base repeated with
substitutions and short insertions and deletions (a collection of genomes),
"versions" a 96-symbol document followed by its edited versions.
"""
import ctypes
import math
import random
import statistics

import numpy as np
import torch

import paper_2512_23314_amd as bt

KIB, MIB = 1 << 10, 1 << 20
ACGT = (65, 67, 71, 84)
# newline and the printable ASCII characters
SYMBOLS = np.concatenate([np.array([10], np.uint8), np.arange(0x20, 0x7F, dtype=np.uint8)])


def _build(name, text, n, tau, leaf, option="plain"):
    return {"name": name, "kind": "build", "text": text, "n": n, "tau": tau, "leaf": leaf,
            "option": option}


def _batch(name, texts, median, spread, tau, leaf):
    return {"name": name, "kind": "batch", "text": "dna", "texts": texts, "median": median,
            "spread": spread, "tau": tau, "leaf": leaf}


def _query(name, text, n, m):
    return {"name": name, "kind": "query", "text": text, "n": n, "m": m, "tau": 4, "leaf": 16}


def listed():
    return [
        # a single short document: launches and read-backs count, not bytes
        _build("build_4k", "dna", 4 * KIB, 2, 16),
        # an ordinary small text, binary splits (16 levels)
        _build("build_1m", "dna", 1 * MIB, 2, 16),
        # the index with rank/select support over a 96-symbol alphabet, odd size
        _build("build_rank_16m", "versions", 16 * MIB + 77, 4, 16, "rank"),
        # a versioned document collection
        _build("build_versions_256m", "versions", 256 * MIB, 4, 16),
        # the largest single text: a collection of genomes
        _build("build_dna_2g", "dna", 2048 * MIB, 4, 16),
        # deep trees, short leaves, a text that ends inside a block
        _build("build_dna_odd", "dna", 100000007, 2, 8),
        # the build for little memory
        _build("build_lean_odd", "versions", 128 * MIB - 12345, 4, 16, "lean"),
        # the smallest trees (unneeded marks taken out)
        _build("build_prune_64m", "versions", 64 * MIB, 4, 16, "prune"),
        # many short documents in one call (a server's small requests)
        _batch("batch_small", 64, 16 * KIB, 1.0, 4, 16),
        # an ordinary batch of uneven texts
        _batch("batch_uneven", 192, 1 * MIB, 1.5, 4, 16),
        # a large batch of queries against a resident tree
        _query("query_1m", "versions", 64 * MIB, 1 << 20),
        # a handful of queries: latency
        _query("query_few", "dna", 1 * MIB, 300),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build", "build", "build", "batch", "query"])
    if kind == "build":
        option = rng.choice(["plain", "plain", "lean", "prune", "rank"])
        top = {"rank": 32 * MIB, "prune": 128 * MIB}.get(option, 320 * MIB)
        c = _build("", rng.choice(["dna", "versions"]), _log_int(rng, 1 * KIB, top),
                   rng.choice([2, 4, 8, 16]), rng.choice([8, 16, 32]), option)
    elif kind == "batch":
        texts = _log_int(rng, 4, 224)
        # at most about 512 MiB in all (the mean of the sizes is below 3.1 medians)
        c = _batch("", texts, _log_int(rng, 2 * KIB, min(2 * MIB, 160 * MIB // texts)),
                   round(rng.uniform(0.0, 1.5), 2), rng.choice([2, 4, 8]), rng.choice([8, 16, 32]))
    else:
        c = _query("", rng.choice(["dna", "versions"]), _log_int(rng, 64 * KIB, 64 * MIB),
                   _log_int(rng, 1, 1 << 20))
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _dna(n, base_len, sub, indel, indel_max, g):
    """A random base repeated to n bytes with substitutions (rate sub) and
    insertions and deletions (rate indel, 1 to indel_max symbols)."""
    dev = g.device
    sym = torch.tensor(ACGT, dtype=torch.uint8, device=dev)
    base = torch.randint(0, 4, (base_len,), generator=g, dtype=torch.uint8, device=dev)
    out = torch.empty(n, dtype=torch.uint8, device=dev)
    at = 0
    step = 64 * MIB
    for lo in range(0, n, step):
        k = min(step, n - lo)
        u = torch.rand(k, generator=g, device=dev)
        where = torch.nonzero(u < indel).flatten()
        size = torch.randint(1, indel_max + 1, (where.numel(),), generator=g, device=dev)
        grow = torch.rand(where.numel(), generator=g, device=dev) < 0.5
        shift = torch.zeros(k + 1, dtype=torch.int32, device=dev)
        shift[where] = torch.where(grow, -size, size).to(torch.int32)
        src = torch.cumsum(shift[:k], 0, dtype=torch.int32)
        last = int(src[-1])
        src += torch.arange(at, at + k, dtype=torch.int32, device=dev)
        idx = base[torch.remainder(src, base_len).long()]
        # inserted symbols are new ones, and so are substituted ones
        edge = torch.zeros(k + 1, dtype=torch.int32, device=dev)
        ins, ends = where[grow], torch.clamp(where[grow] + size[grow], max=k)
        edge.index_add_(0, ins, torch.ones_like(ins, dtype=torch.int32))
        edge.index_add_(0, ends, -torch.ones_like(ends, dtype=torch.int32))
        new = torch.nonzero((torch.cumsum(edge[:k], 0) > 0) | (u > 1.0 - sub)).flatten()
        turn = torch.randint(1, 4, (new.numel(),), generator=g, dtype=torch.uint8, device=dev)
        idx[new] = (idx[new] + turn) % 4
        out[lo:lo + k] = sym[idx.long()]
        at = (at + k + last) % base_len
    return out


def _versions(n, seed):
    """A document of at most 256 KiB over 96 symbols (an order-2 chain) and its
    versions, each with edits (substituted, inserted or deleted runs of 1 to 64
    symbols, one per 2000 symbols) of the version before."""
    r = np.random.default_rng(seed)
    s = SYMBOLS.size
    base_len = max(64, min(256 * KIB, n // 16))
    rank = np.argsort(r.random((s * s, s)), axis=1).astype(np.uint8)
    w = np.cumsum(1.0 / np.arange(1, s + 1) ** 1.5)
    pick = np.minimum(np.searchsorted(w / w[-1], r.random(base_len + 8 * KIB)), s - 1).tolist()
    rows = rank.tolist()
    chain, a, b = [], 0, 0
    for p in pick:
        a, b = b, rows[a * s + b][p]
        chain.append(b)
    chain = SYMBOLS[np.array(chain, np.uint8)]
    cur, pool = chain[:base_len], chain[base_len:]
    parts, have = [], 0
    while have < n:
        parts.append(cur)
        have += cur.size
        k = int(round(cur.size / 2000))
        pos = np.sort(r.integers(0, cur.size, k)).tolist()
        size = r.integers(1, 65, k).tolist()
        op = r.integers(0, 3, k).tolist()
        new = r.integers(0, pool.size - 64, k).tolist()
        pieces, prev = [], 0
        for p, l, o, q in zip(pos, size, op, new):
            if p < prev:
                continue
            pieces.append(cur[prev:p])
            if o < 2:
                pieces.append(pool[q:q + l])
            prev = p if o == 1 else min(cur.size, p + l)
        pieces.append(cur[prev:])
        cur = np.concatenate(pieces)
    return torch.from_numpy(np.concatenate(parts)[:n]).cuda()


def _sizes(case):
    """A batch's text sizes: lognormal, at even quantiles, in a fixed shuffled order."""
    q = statistics.NormalDist()
    t = case["texts"]
    sizes = [case["median"] * math.exp(case["spread"] * q.inv_cdf((i + 0.5) / t)) for i in range(t)]
    random.Random(t).shuffle(sizes)
    return [min(max(int(round(x)), 256), 32 * MIB) for x in sizes]


def _text(kind, n, seed, rate=1e-3):
    if kind == "versions":
        return _versions(n, seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return _dna(n, max(16, min(8 * MIB, n // 16)), rate, rate / 10, 20 if n > 16 * MIB else 8, g)


def _options(case):
    opt = case.get("option", "plain")
    return {"tau": case["tau"], "leaf_len": case["leaf"], "sigma": 96 if case["text"] == "versions" else 4,
            "rank_select": opt == "rank" or case["kind"] == "query", "prune": opt == "prune",
            "lean": opt == "lean"}


def _queries(text, m, seed):
    """Uniform positions, characters drawn from the text, ranks up to about
    their count."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    n = text.numel()
    pos = torch.randint(0, n, (m,), generator=g, device="cuda")
    ch = text[torch.randint(0, n, (m,), generator=g, device="cuda")].contiguous()
    count = torch.bincount(text[:64 * MIB].int(), minlength=256)
    k = 1 + (torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * count[ch.long()]).long()
    return {"pos": pos.to(torch.uint64), "ch": ch, "k": k.to(torch.uint64)}


def prepare(case, seed):
    s = {"case": case, "opt": _options(case)}
    if case["kind"] == "batch":
        sizes = _sizes(case)
        s["offsets"] = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
        rates = np.random.default_rng(seed).uniform(1e-4, 1e-2, case["texts"])
        s["text"] = torch.cat([_text("dna", int(n), seed * 1009 + i, float(rates[i]))
                               for i, n in enumerate(sizes)])
    else:
        s["text"] = _text(case["text"], case["n"], seed)
    s["ctx"] = bt.Context(0)
    if case["kind"] != "query":
        s["out"] = _buffers(case)
    if case["kind"] == "query":
        s.update(_queries(s["text"], case["m"], seed))
        s["tree"] = s["ctx"].build(s["text"], **s["opt"])
    elif s["opt"]["rank_select"]:
        s.update(_queries(s["text"], min(1 << 16, case["n"]), seed))
    return s


# ---------------------------------------------------------------- one pass

def _buffers(case):
    """Room for the trees' read-out: level sizes, marks (64-bit words) and
    pointers (target block, offset) on the GPU, leaf bytes in pinned host memory."""
    marks = ptrs = total = levels = 0
    for n in _sizes(case) if case["kind"] == "batch" else [case["n"]]:
        b, h = case["leaf"], 1
        while b <= n // case["tau"]:
            b *= case["tau"]
            h += 1
            marks += n // b // 64 + 1
            ptrs += n // b + 1
        levels += h
        total += n + case["leaf"]
    # above 1 GiB at most a quarter of the text is leaves (a pass on one with more fails)
    if total > 1024 * MIB:
        total //= 4
    dev = {"dtype": torch.int64, "device": "cuda"}
    return {"sizes": np.zeros((levels, 3), np.int64), "marks": torch.zeros(marks, **dev),
            "block": torch.zeros(ptrs, **dev), "off": torch.zeros(ptrs, **dev),
            "leaves": torch.zeros(total, dtype=torch.uint8, pin_memory=True)}


def _read_out(ctx, trees, out):
    """Every tree's levels one after another, into the state's buffers."""
    lib = bt.lib()
    stream = ctx.stream.cuda_stream
    sizes, nb = out["sizes"], ctypes.c_uint64()
    pm, pb, po, pl = (out[k].data_ptr() for k in ("marks", "block", "off", "leaves"))
    end = pl + out["leaves"].numel()
    k = 0
    for t in trees:
        h = t.height
        for l in range(1, h + 1):
            sizes[k] = b, c, u = t.level_info(l)
            k += 1
            if l == h:
                break
            if lib.bt_level_copy_async(t.h, l, pm, pb, po, stream):
                raise RuntimeError("bt_level_copy_async")
            pm += (c + 63) // 64 * 8
            pb += 8 * u
            po += 8 * u
        lib.bt_leaves_size(t.h, ctypes.byref(nb))
        if pl + nb.value > end or lib.bt_leaves_copy(t.h, pl):
            raise RuntimeError("bt_leaves_copy")
        pl += nb.value
    return dict(out)


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["kind"] == "query":
        t = state["tree"]
        return {"access": t.access(state["pos"]), "rank": t.rank(state["ch"], state["pos"]),
                "select": t.select(state["ch"], state["k"])}
    if case["kind"] == "batch":
        trees = ctx.build_batch(state["text"], state["offsets"], **state["opt"])
        out = _read_out(ctx, trees, state["out"])
        bt.free_trees(trees)
        return out
    tree = ctx.build(state["text"], **state["opt"])
    out = _read_out(ctx, [tree], state["out"])
    if state["opt"]["rank_select"]:
        out["rank"] = tree.rank(state["ch"], state["pos"])
        out["select"] = tree.select(state["ch"], state["k"])
    tree.free()
    return out


def work(case):
    """Bytes a pass cannot do without.  A build reads its text; a tree's size
    depends on the text (far below the text's for repetitive ones) and is not
    counted.  A query batch reads its positions, characters and ranks and writes
    its answers."""
    if case["kind"] == "query":
        return {"bytes": case["m"] * ((8 + 1) + (8 + 1 + 8) + (8 + 1 + 8)), "flops": 0}
    if case["kind"] == "batch":
        return {"bytes": sum(_sizes(case)), "flops": 0}
    return {"bytes": case["n"], "flops": 0}


def exact(case, seed):
    """The answers of a query pass by counting; a tree has no value that is
    quicker to state than to build."""
    if case["kind"] != "query":
        return None
    text = _text(case["text"], case["n"], seed)
    q = _queries(text, case["m"], seed)
    text = text.cpu().numpy()
    pos = q["pos"].to(torch.int64).cpu().numpy()
    ch, k = q["ch"].cpu().numpy(), q["k"].to(torch.int64).cpu().numpy()
    rank, select = np.zeros(pos.size, np.uint64), np.zeros(pos.size, np.uint64)
    for c in np.unique(ch):
        at = np.flatnonzero(text == c)
        of = ch == c
        rank[of] = np.searchsorted(at, pos[of])
        select[of] = at[k[of] - 1]
    return {"access": torch.from_numpy(text[pos]), "rank": torch.from_numpy(rank),
            "select": torch.from_numpy(select)}
