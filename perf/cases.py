"""Timed cases of the static index: what a program does with it, by size.

Every case is one call sequence through the package's public entry points.
Indexes take the form the tuned table gives for their layout and size, as a
program that asks `autotune.choose` (or, in a batch, `autotune.batch_form`)
gets it.  Keys, row IDs and queries are made on the GPU from the seed.

Fields of a case: `op`, then the sizes and options of that operation:
  point        m lookups (share `hit` of them hits, Zipf exponent `zipf`, 0 =
               uniform) in an index of n keys, layout `form`
  range        m ranges of 1..`width` matches (all `width` when `fixed`)
  build        sort and lay out n pairs, then read the layout back
  merge        a new index over n sorted pairs and m new ones, read back
  learn        train the rank model, read its leaf table, first lookups
  batch_point  point lookups over `count` indexes in one launch
  batch_mixed  points and ranges over `count` indexes in one stream
`bits` is the key width; `dist` the key distribution (uniform, or a mixture
of 64 lognormal clusters for 64-bit keys).
"""
import math

import torch

import paper_2506_01576_amd as idx
from paper_2506_01576_amd import Batch, Index, autotune, learn_batch


def listed():
    return [
        # a service answering one small request from a cache-resident index: launch latency
        {"name": "point_u32_ebs_small", "op": "point", "form": "ebs", "bits": 32, "n": 4096, "m": 1000, "hit": 0.5,
         "zipf": 0.0, "dist": "uniform"},
        # the plain sorted array of 2^16 keys under 2^20 lookups, half of them misses
        {"name": "point_u32_bs_2p16", "op": "point", "form": "bs", "bits": 32, "n": 1 << 16, "m": 1 << 20, "hit": 0.5,
         "zipf": 0.0, "dist": "uniform"},
        # full-scale bulk probes (a join's probe side), one case per form
        {"name": "point_u64_bs_2p26", "op": "point", "form": "bs", "bits": 64, "n": 1 << 26, "m": 1 << 27, "hit": 1.0,
         "zipf": 0.0, "dist": "uniform"},
        {"name": "point_u64_eks_2p26", "op": "point", "form": "eks", "bits": 64, "n": 1 << 26, "m": 1 << 27,
         "hit": 1.0, "zipf": 0.0, "dist": "uniform"},
        {"name": "point_u64_learned_2p26", "op": "point", "form": "learned", "bits": 64, "n": 1 << 26, "m": 1 << 27,
         "hit": 1.0, "zipf": 0.0, "dist": "uniform"},
        # bulk range scans of 16 rows each on the sorted array
        {"name": "range_u64_bs_2p26", "op": "range", "form": "bs", "bits": 64, "n": 1 << 26, "m": 1 << 24,
         "width": 16, "fixed": True},
        # uneven ranges of 1..256 rows on a mid-sized k-ary tree of odd size
        {"name": "range_u32_eks_10m", "op": "range", "form": "eks", "bits": 32, "n": 10000019, "m": 1000003,
         "width": 256, "fixed": False},
        # (re)building the index over a full column
        {"name": "build_u64_eks_2p26", "op": "build", "form": "eks", "bits": 64, "n": 1 << 26, "dist": "uniform"},
        # the read-mostly update: a small batch of new rows into a sorted index, odd sizes
        {"name": "merge_u32_bs_1m", "op": "merge", "form": "bs", "bits": 32, "n": 1000003, "m": 50021,
         "dist": "uniform"},
        # training the rank model over a full column, leaf lines included
        {"name": "learn_u64_2p26", "op": "learn", "bits": 64, "n": 1 << 26, "leaves": 1 << 24, "lines": True,
         "dist": "uniform"},
        # many indexes of 2^6..2^22 keys with uneven batches, replayed from a graph
        {"name": "batch_point_u32_512", "op": "batch_point", "bits": 32, "count": 512, "graph": True, "salt": 1},
        # a mixed stream (70% points with 10% misses, 30% ranges of 1..256 rows) over learned indexes
        {"name": "batch_mixed_u64_64", "op": "batch_mixed", "form": "learned", "bits": 64, "count": 64, "salt": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["point"] * 5 + ["range"] * 3 + ["build", "build", "merge", "learn", "learn", "batch_point",
                                                     "batch_mixed"])
    bits = rng.choice([32, 64])
    dist = rng.choice(["uniform", "uniform", "lognormal"]) if bits == 64 else "uniform"
    if op == "point":
        n = _log_int(rng, 1 << 12, 1 << 26)
        return {"op": op, "form": rng.choice(["bs", "ebs", "eks", "learned"]), "bits": bits, "n": n,
                "m": _log_int(rng, 500, 1 << 27), "hit": rng.choice([1.0, 0.9, 0.5]),
                "zipf": rng.choice([0.0, 0.0, 0.5, 1.1]), "dist": dist}
    if op == "range":
        n = _log_int(rng, 1 << 16, 1 << 26)
        width = rng.choice([1, 16, 16, 64, 256])
        return {"op": op, "form": rng.choice(["bs", "ebs", "eks", "learned"]), "bits": bits, "n": n,
                "m": min(_log_int(rng, 500, 1 << 24), (1 << 28) // width), "width": width,
                "fixed": rng.choice([True, False])}
    if op == "build":
        return {"op": op, "form": rng.choice(["bs", "ebs", "eks"]), "bits": bits, "n": _log_int(rng, 1000, 1 << 26),
                "dist": dist}
    if op == "merge":
        n = _log_int(rng, 1 << 16, 1 << 25)
        return {"op": op, "form": rng.choice(["bs", "ebs", "eks"]), "bits": bits, "n": n,
                "m": _log_int(rng, 1000, max(2000, n // 8)), "dist": dist}
    if op == "learn":
        n = _log_int(rng, 1 << 16, 1 << 26)
        per_leaf = rng.choice([4, 16, 64])
        return {"op": op, "bits": bits, "n": n, "leaves": max(1, n // per_leaf), "lines": per_leaf == 4, "dist": dist}
    if op == "batch_point":
        return {"op": op, "bits": bits, "count": rng.randint(100, 512), "graph": rng.choice([True, False]),
                "salt": rng.randrange(1 << 20)}
    return {"op": op, "form": rng.choice(["learned", "eks"]), "bits": 64, "count": rng.randint(16, 64),
            "salt": rng.randrange(1 << 20)}


# ------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed & 0x7FFFFFFFFFFFFFFF)
    return g


def _mixed_key(seed, w, x):
    """A seeded bijection of [0, 2^w) applied to the int64 tensor x: x -> key."""
    mask = (1 << w) - 1
    g = torch.Generator().manual_seed(seed & 0x7FFFFFFFFFFFFFFF)
    for shift in (w // 2, w // 3 + 1):
        mul, add = (int(v) for v in torch.randint(0, 1 << 62, (2,), generator=g))
        x = (x * (mul | 1) + (add & mask)) & mask
        x = x ^ (x >> shift)
    return x


def _stored(keys, bits):
    """Key values (non-negative int64) as the index takes them."""
    return keys if bits == 64 else torch.where(keys >= 1 << 31, keys - (1 << 32), keys).to(torch.int32)


def _values(keys, bits):
    """The unsigned values of stored keys, as int64 (64-bit keys are below 2^63 here)."""
    return keys if bits == 64 else keys.to(torch.int64) & 0xFFFFFFFF


def _key_set(case, seed, g):
    """n distinct keys in insertion order, and miss(count): keys not in the set."""
    n, bits = case["n"], case["bits"]
    if case.get("dist", "uniform") == "lognormal":
        mu = 20 + 30 * torch.rand(64, generator=g, device="cuda", dtype=torch.float64)
        sigma = 0.5 + 1.5 * torch.rand(64, generator=g, device="cuda", dtype=torch.float64)
        keys, drawn = None, n + n // 8 + 1024
        while keys is None or len(keys) < n:
            c = torch.randint(0, 64, (drawn,), generator=g, device="cuda")
            z = torch.randn(drawn, generator=g, device="cuda", dtype=torch.float64)
            keys = torch.unique(torch.exp(mu[c] + sigma[c] * z).clamp_(max=9.2e18).to(torch.int64))
            drawn *= 2
        keys = keys[torch.randperm(len(keys), generator=g, device="cuda")[:n]].contiguous()

        def miss(count):
            return torch.randint(0, 1 << 62, (count,), generator=g, device="cuda") * 2
        return keys, miss
    w = 32 if bits == 32 else 63
    keys = _mixed_key(seed, w, torch.arange(n, device="cuda", dtype=torch.int64))

    def miss(count):
        return _mixed_key(seed, w, torch.randint(n, (1 << w) - 1, (count,), generator=g, device="cuda"))
    return keys, miss


def _point_queries(keys, miss, m, hit, zipf, g):
    n = len(keys)
    u = torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
    if zipf == 0.0:
        at = (u * n).to(torch.int64)
    else:  # bounded Zipf by inversion of its continuous distribution
        e = 1.0 - zipf
        at = torch.pow((float(n + 1) ** e - 1.0) * u + 1.0, 1.0 / e).to(torch.int64) - 1
    del u
    q = keys[at.clamp_(0, n - 1)]
    if hit < 1.0:
        out = torch.rand(m, generator=g, device="cuda") >= hit
        q[out] = miss(int(out.sum()))
    return q


def _ranges(skeys, m, width, fixed, g):
    """m ranges over the ascending keys: (lo, hi, matches of each); uneven ones take every width equally often."""
    n = len(skeys)
    if fixed:
        c = torch.full((m,), min(width, n), device="cuda", dtype=torch.int64)
    else:
        c = 1 + torch.randperm(m, generator=g, device="cuda") % min(width, n)
    r = (torch.rand(m, generator=g, device="cuda", dtype=torch.float64) * (n - c + 1)).to(torch.int64)
    r = torch.minimum(r, n - c)
    return skeys[r], skeys[r + c - 1], c


def _rows(n):
    return torch.arange(n, device="cuda", dtype=torch.int32)


def _tuned_index(keys, rows, bits, form):
    """An index in the tuned form of its layout and size."""
    layout, k, aos, params = autotune.choose(len(keys), bits, form)
    if layout != "learned":
        ix = Index(keys, rows, layout=layout, k=k, aos=aos)
        ix.set_params(**params)
        return ix
    leaves = params.pop("leaves")
    ix = Index(keys, rows, layout="bs", aos=aos)
    ix.set_params(**params)
    ix.learn(leaves, 2)
    return ix


def _point_inputs(case, seed):
    g = _gen(seed)
    keys, miss = _key_set(case, seed, g)
    q = _point_queries(keys, miss, case["m"], case["hit"], case["zipf"], g)
    return _stored(keys, case["bits"]), _stored(q, case["bits"])


def _range_inputs(case, seed):
    g = _gen(seed)
    keys, _ = _key_set(case, seed, g)
    lo, hi, c = _ranges(torch.sort(keys)[0], case["m"], case["width"], case["fixed"], g)
    return _stored(keys, case["bits"]), _stored(lo, case["bits"]), _stored(hi, case["bits"]), int(c.sum())


def _batch_sizes(case, seed):
    """Sizes and lookup counts of a batch's indexes (the case's own, the same for every seed)."""
    g = torch.Generator().manual_seed(case["salt"])
    lo, hi, qlo, qhi = (6, 22, 0, 16) if case["op"] == "batch_point" else (16, 24, 10, 18)
    u = torch.rand(2, case["count"], generator=g, dtype=torch.float64)
    n = torch.pow(2.0, lo + (hi - lo) * u[0]).to(torch.int64).tolist()
    m = torch.pow(2.0, qlo + (qhi - qlo) * u[1]).to(torch.int64).tolist()
    return n, m


def _offsets(counts):
    return torch.tensor([0] + counts, dtype=torch.int64).cumsum(0).cuda()


# ------------------------------------------------------------------ protocol

def prepare(case, seed):
    op, bits = case["op"], case["bits"]
    if op == "point":
        keys, q = _point_inputs(case, seed)
        return {"op": op, "ix": _tuned_index(keys, _rows(case["n"]), bits, case["form"]), "q": q}
    if op == "range":
        keys, lo, hi, total = _range_inputs(case, seed)
        return {"op": op, "ix": _tuned_index(keys, _rows(case["n"]), bits, case["form"]), "lo": lo, "hi": hi,
                "total": total}
    if op == "build":
        keys = _stored(_key_set(case, seed, _gen(seed))[0], bits)
        return {"op": op, "keys": keys, "rows": _rows(case["n"]), "form": case["form"]}
    if op == "merge":
        n, m = case["n"], case["m"]
        keys = _stored(_key_set(dict(case, n=n + m), seed, _gen(seed))[0], bits)
        rows = _rows(n + m)
        return {"op": op, "ix": Index(keys[:n], rows[:n], layout="bs"), "keys": keys[n:].contiguous(),
                "rows": rows[n:].contiguous(), "form": case["form"]}
    if op == "learn":
        g = _gen(seed)
        keys, miss = _key_set(case, seed, g)
        q = _point_queries(keys, miss, 1 << 16, 0.5, 0.0, g)
        ix = Index(_stored(keys, bits), _rows(case["n"]), layout="bs")
        if case["lines"]:
            ix.set_params(leaf_lines=1)
        return {"op": op, "ix": ix, "leaves": case["leaves"], "q": _stored(q, bits)}
    sizes, counts = _batch_sizes(case, seed)
    g = _gen(seed)
    members, los, his, kinds, total = [], [], [], [], 0
    for j, (n, m) in enumerate(zip(sizes, counts)):
        one = {"n": n, "bits": bits, "dist": "lognormal" if op == "batch_mixed" and j % 2 else "uniform"}
        keys, miss = _key_set(one, seed * 8191 + j, g)
        rows = _rows(n)
        if op == "batch_point":
            los.append(_stored(_point_queries(keys, miss, m, 0.8, 0.0, g), bits))
            members.append(autotune.build_form(_stored(keys, bits), rows, autotune.batch_form(n, bits)))
            continue
        lo = _point_queries(keys, miss, m, 0.9, 0.0, g)
        hi = lo.clone()
        kind = torch.randperm(m, generator=g, device="cuda") < 3 * m // 10
        rl, rh, c = _ranges(torch.sort(keys)[0], 3 * m // 10, 256, False, g)
        lo[kind], hi[kind] = rl, rh
        total += int(c.sum())
        los.append(lo)
        his.append(hi)
        kinds.append(kind.to(torch.uint8))
        members.append(Index(keys, rows, layout="bs") if case["form"] == "learned"
                       else Index(keys, rows, layout="eks", k=17))
    if op == "batch_mixed" and case["form"] == "learned":
        learn_batch(members, [max(1, n // 64) for n in sizes], 2)
    state = {"op": op, "batch": Batch(members), "lo": torch.cat(los), "offsets": _offsets(counts)}
    if op == "batch_point":
        return dict(state, graph=case["graph"], out=torch.empty(sum(counts), dtype=torch.int32, device="cuda"))
    return dict(state, hi=torch.cat(his), kind=torch.cat(kinds), total=total)


def run(state):
    op = state["op"]
    if op == "point":
        return state["ix"].point(state["q"])
    if op == "range":
        return state["ix"].range(state["lo"], state["hi"], capacity=state["total"])
    if op == "build":
        with Index(state["keys"], state["rows"], layout=state["form"], k=9) as ix:
            return ix.export()
    if op == "merge":
        with state["ix"].merge(state["keys"], state["rows"], layout=state["form"], k=9) as ix:
            return ix.export()
    if op == "learn":
        ix = state["ix"]
        stats = ix.learn(state["leaves"], 2)
        table = ix.learn_export()
        b0, b1 = (table[:, j].view(torch.float32) for j in (4, 5))
        return {"feature": stats["feature"], "root_loss": stats["root_loss"], "leaf_loss": stats["leaf_loss"],
                "mean_window": stats["mean_window"], "max_window": stats["max_window"], "b0": b0, "b1": b1,
                "first": table[:, :4], "errors": table[:, 6:], "ids": ix.point(state["q"])}
    if op == "batch_point":
        return state["batch"].point(state["lo"], state["offsets"], state["out"], graph=state["graph"])
    return state["batch"].mixed(state["lo"], state["hi"], state["kind"], state["offsets"], capacity=state["total"])


def work(case):
    """Inputs read once, outputs written once, and the index entries that the lookups meet read once each."""
    op, entry = case["op"], case["bits"] // 8 + 4
    key = entry - 4
    n, m = case.get("n", 0), case.get("m", 0)
    if op == "point":
        return {"bytes": m * entry + min(n, m) * entry, "flops": 0}
    if op == "range":
        total = m * (case["width"] if case["fixed"] else (case["width"] + 1) / 2)
        return {"bytes": m * (2 * key + 8) + min(n, 2 * m) * key + 8 * total, "flops": 0}
    if op == "build":  # the pairs in, the layout out, and its copy for the caller
        return {"bytes": 4 * n * entry, "flops": 0}
    if op == "merge":
        return {"bytes": 4 * (n + m) * entry, "flops": 0}
    if op == "learn":  # the keys (row IDs too with lines) in, leaf records (and lines) out, the table's copy
        return {"bytes": n * (entry if case["lines"] else key) + case["leaves"] * (224 if case["lines"] else 96),
                "flops": 0}
    sizes, counts = _batch_sizes(case, 0)
    touched = sum(min(a, b) for a, b in zip(sizes, counts))
    if op == "batch_point":
        return {"bytes": sum(counts) * entry + touched * entry, "flops": 0}
    # per query both bounds, its kind, an answer and an offset; per matched row its ID read and written
    return {"bytes": sum(counts) * (2 * key + 13) + touched * key + 8 * 128.5 * 0.3 * sum(counts), "flops": 0}


# ------------------------------------------------------------ 64-bit answers

def _sorted_pairs(keys, bits):
    return torch.sort(_values(keys, bits))


def exact(case, seed):
    op, bits = case["op"], case["bits"]
    if op == "point":
        keys, q = _point_inputs(case, seed)
        sk, order = _sorted_pairs(keys, bits)
        q = _values(q, bits)
        at = torch.searchsorted(sk, q).clamp_(max=len(sk) - 1)
        return torch.where(sk[at] == q, order[at], -1).to(torch.int32)
    if op == "range":
        keys, lo, hi, total = _range_inputs(case, seed)
        sk, order = _sorted_pairs(keys, bits)
        first = torch.searchsorted(sk, _values(lo, bits))
        counts = torch.searchsorted(sk, _values(hi, bits), right=True) - first
        offsets = torch.zeros(case["m"] + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(counts, 0, out=offsets[1:])
        at = torch.arange(total, device="cuda") + torch.repeat_interleave(first - offsets[:-1], counts)
        return offsets, order[at].to(torch.int32)
    if op in ("build", "merge") and case["form"] == "bs":
        keys = _key_set(dict(case, n=case["n"] + case.get("m", 0)), seed, _gen(seed))[0]
        sk, order = torch.sort(keys)
        return _stored(sk, bits), order.to(torch.int32)
    if op == "learn" and case.get("dist") == "uniform":
        return _exact_model(torch.sort(_key_set(case, seed, _gen(seed))[0])[0], case["leaves"])
    return None


def _fit(n, sx, sxx, sy, sxy):
    """Least squares of y on x from their sums: (intercept, slope)."""
    det = n * sxx - sx * sx
    line = (n >= 2) & (det > 1e-12 * n * sxx)
    det = torch.where(line, det, torch.ones_like(det))
    slope = torch.where(line, (n * sxy - sx * sy) / det, torch.zeros_like(det))
    mean = sy / n.clamp(min=1)
    return torch.where(line, (sxx * sy - sx * sxy) / det, mean), slope


def _exact_model(keys, leaves):
    """The two-stage fit of rank on key: a line over the key scaled to [0, 1], whose (32-bit) weights assign the
    keys to leaves, and a line per leaf over the offset from its first key."""
    n = len(keys)
    rank = torch.arange(n, device="cuda", dtype=torch.float64)
    target = (rank * (leaves / n)).to(torch.float32)
    x = keys.to(torch.float32) * 2.0 ** -64
    xd = x.double()
    count = torch.tensor(float(n), device="cuda", dtype=torch.float64)
    a0 = a1 = torch.zeros((), device="cuda")
    for _ in range(2):  # the second step corrects the first one's rounding
        r = (target - (a1 * x + a0)).double()
        d0, d1 = _fit(count, xd.sum(), (xd * xd).sum(), r.sum(), (r * xd).sum())
        a0, a1 = (a0.double() + d0).float(), (a1.double() + d1).float()
    root_loss = float((a1 * x + a0 - target).double().square().sum())
    del xd, target
    leaf = (a1 * x + a0).clamp(0, leaves - 1).to(torch.int64)
    size = torch.bincount(leaf, minlength=leaves)
    base = size.cumsum(0) - size
    y = rank - base[leaf]
    d = (keys - keys[base.clamp(max=n - 1)][leaf]).double()

    def per_leaf(v):
        return torch.zeros(leaves, dtype=torch.float64, device="cuda").index_add_(0, leaf, v)
    b0, b1 = _fit(size.double(), per_leaf(d), per_leaf(d * d), per_leaf(y), per_leaf(d * y))
    return {"feature": None, "root_loss": root_loss, "leaf_loss": None, "mean_window": None, "max_window": None,
            "b0": b0, "b1": b1, "first": None, "errors": None, "ids": None}
