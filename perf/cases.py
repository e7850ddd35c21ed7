"""Performance cases of the FSI operator and of the tree-ensemble value function.

Each case is one call, or one short chain of calls, that a user of the package
makes: plans and forests are built once, inputs and outputs are device
buffers, and a pass is the apply itself. Inputs are the games the repository
works with (tree ensembles explained at one point against background points,
and planted sparse games), made from the seed with plain torch.
"""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
import torch

from paper_2601_01903_amd import BatchPlan, Forest, Plan

DEV = "cuda"
TORCH_DTYPE = {"f32": torch.float32, "f64": torch.float64}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: 8 players, pairs, one explained instance (latency)
        {"name": "single_d8_l2_f64", "kind": "single", "d": 8, "l": 2, "dtype": "f64",
         "precision": "auto", "index": "fsi", "game": "planted"},
        # a 14-feature tree model explained in double precision, triples
        {"name": "single_d14_l3_f64", "kind": "single", "d": 14, "l": 3, "dtype": "f64",
         "precision": "auto", "index": "fsi", "game": "tree"},
        # 20 features, order 4, one instance at a time
        {"name": "single_d20_l4_f32", "kind": "single", "d": 20, "l": 4, "dtype": "f32",
         "precision": "auto", "index": "fsi", "game": "tree"},
        # many instances of uneven size in one batch (d 8 to 20, orders 1 to 4)
        {"name": "ragged_512_f32", "kind": "ragged", "n": 512, "dlo": 8, "dhi": 20, "llo": 1,
         "lhi": 4, "dtype": "f32", "precision": "auto", "index": "fsi"},
        # throughput: 256 instances of 20 features, order 4, default FP32 form
        {"name": "batch_256_d20_l4_f32", "kind": "batch", "n": 256, "d": 20, "l": 4,
         "dtype": "f32", "precision": "auto", "index": "fsi"},
        # the same in double precision, a smaller batch, Shapley interaction index
        {"name": "batch_48_d20_l3_f64_sii", "kind": "batch", "n": 48, "d": 20, "l": 3,
         "dtype": "f64", "precision": "auto", "index": "sii"},
        # one very large instance: outputs past one workgroup's accumulators
        {"name": "single_d27_l4_f32", "kind": "single", "d": 27, "l": 4, "dtype": "f32",
         "precision": "auto", "index": "fsi", "game": "planted"},
        # orders above 4 (generic kernels): a few instances at order 6
        {"name": "batch_8_d18_l6_f32", "kind": "batch", "n": 8, "d": 18, "l": 6,
         "dtype": "f32", "precision": "auto", "index": "fsi"},
        # the Moebius transform alone, of a copy of the values
        {"name": "mobius_d24_f64", "kind": "mobius", "d": 24, "dtype": "f64"},
        # value function of a forest at 20 features, one background point
        {"name": "forest_walk_d20_bg1_f32", "kind": "forest", "d": 20, "trees": 200, "depth": 6,
         "n_bg": 1, "method": "walk", "dtype": "f32"},
        # interventional value function over 100 background points, 14 features
        {"name": "forest_walk_d14_bg100_f64", "kind": "forest", "d": 14, "trees": 50, "depth": 4,
         "n_bg": 100, "method": "walk", "dtype": "f64"},
        # the Moebius route to v, 100 background points, then the operator on v
        {"name": "forest_mobius_fsi_d20_bg100", "kind": "forest_fsi", "d": 20, "trees": 200,
         "depth": 6, "n_bg": 100, "l": 3, "dtype": "f64"},
    ]


def _logint(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["single", "single", "ragged", "batch", "batch", "high", "mobius", "forest",
                       "forest", "forest_fsi"])
    dtype = rng.choice(["f32", "f64"])
    index = rng.choice(["fsi", "fsi", "fsi", "stii", "sii", "ksii", "bii"])
    prec = "auto"
    if dtype == "f32":
        prec = rng.choice(["auto", "auto", "auto", "f32", "f32_compensated"])
    if kind == "single":
        d = rng.randint(5, 26 if dtype == "f32" else 25)
        return {"kind": "single", "d": d, "l": rng.randint(1, min(4, d)), "dtype": dtype,
                "precision": prec, "index": index, "game": rng.choice(["tree", "planted"])}
    if kind == "ragged":
        dlo = rng.randint(6, 14)
        dhi = rng.randint(dlo + 2, 19)
        llo = rng.randint(1, 3)
        return {"kind": "ragged", "n": _logint(rng, 12, 400), "dlo": dlo, "dhi": dhi, "llo": llo,
                "lhi": rng.randint(llo + 1, 4), "dtype": dtype, "precision": prec, "index": index}
    if kind == "batch":
        d = rng.randint(9, 21)
        n = max(1, min(_logint(rng, 3, 900), (1 << (26 if dtype == "f32" else 25)) >> d))
        return {"kind": "batch", "n": n, "d": d, "l": rng.randint(1, 4), "dtype": dtype,
                "precision": prec, "index": index}
    if kind == "high":
        l = rng.randint(5, 8)
        d = rng.randint(l + 1, 16)
        return {"kind": "batch", "n": _logint(rng, 1, 12), "d": d, "l": l, "dtype": dtype,
                "precision": "auto", "index": index}
    if kind == "mobius":
        return {"kind": "mobius", "d": rng.randint(10, 24), "dtype": dtype}
    if kind == "forest":
        d = rng.randint(6, 17)
        n_bg = _logint(rng, 1, 100)
        trees = _logint(rng, 10, 200)
        depth = rng.randint(3, 6)
        while (trees * n_bg * depth) << d > 1 << 31:
            if n_bg > 1:
                n_bg = max(1, n_bg // 2)
            else:
                d -= 1
        return {"kind": "forest", "d": d, "trees": trees, "depth": depth, "n_bg": n_bg,
                "method": rng.choice(["walk", "walk", "mobius"]), "dtype": dtype}
    return {"kind": "forest_fsi", "d": rng.randint(8, 20), "trees": _logint(rng, 10, 200),
            "depth": rng.randint(3, 6), "n_bg": _logint(rng, 1, 100), "l": rng.randint(1, 4),
            "dtype": dtype}


# --------------------------------------------------------------------- inputs
def _grid(x):
    """Rounds to multiples of 2^-40: sums of a few thousand such values are
    exact in FP64, so a game does not depend on the order of its sums."""
    return np.round(np.asarray(x) * 2.0 ** 40) * 2.0 ** -40


def _forest_params(rng, d, trees, depth):
    inner = (1 << depth) - 1
    return {"feat": rng.integers(0, d, size=(trees, inner)),
            "thr": rng.random((trees, inner)),
            "leaf": _grid(rng.standard_normal((trees, inner + 1)))}


def _tree_coeffs(p, x, b, depth):
    """Moebius coefficients of sum_k f_k (coalition masks, values): each leaf's
    indicator is a product over its path's features."""
    trees, leaves = p["leaf"].shape
    leaf = np.arange(leaves)
    node = np.zeros(leaves, dtype=np.int64)
    shape = (trees, leaves)
    seen = np.zeros(shape, dtype=np.int64)
    abad = np.zeros(shape, dtype=np.int64)
    bbad = np.zeros(shape, dtype=np.int64)
    feats = []
    for lv in range(depth):
        go = (leaf >> (depth - 1 - lv)) & 1
        f, th = p["feat"][:, node], p["thr"][:, node]
        bit = np.int64(1) << f
        seen |= bit
        abad |= np.where((x[f] >= th) != go, bit, 0)
        bbad |= np.where((b[f] >= th) != go, bit, 0)
        feats.append(bit)
        node = 2 * node + 1 + go
    ok = (bbad & abad) == 0
    inc, free = bbad[ok], (seen & ~bbad & abad)[ok]
    val = p["leaf"][ok]
    bits = np.stack([f[ok] for f in feats], axis=1)       # (paths, depth)
    use = (bits & free[:, None]) != 0
    for i in range(1, depth):                              # first occurrence of a feature only
        for j in range(i):
            use[:, i] &= ~((bits[:, i] == bits[:, j]) & use[:, j])
    masks, vals = [inc], [val]
    for i in range(depth):
        m, v = np.concatenate(masks), np.concatenate(vals)
        sel = np.tile(use[:, i], len(m) // len(inc))
        bi = np.tile(bits[:, i], len(m) // len(inc))
        masks.append(np.where(sel, m | bi, m))
        vals.append(np.where(sel, -v, 0.0))
    m, v = np.concatenate(masks), np.concatenate(vals)
    nz = v != 0
    return m[nz], v[nz]


def _planted_coeffs(rng, d, terms, kmax):
    size = rng.integers(1, min(kmax, d) + 1, size=terms)
    perm = np.argsort(rng.random((terms, d)), axis=1)
    take = np.arange(d)[None, :] < size[:, None]
    masks = (np.where(take, np.int64(1) << perm, 0)).sum(axis=1)
    return masks, _grid(rng.standard_normal(terms))


def _zeta_(a, d):
    """Subset sums over the last axis (2^d), in place."""
    flat = a.view(-1, 1 << d)
    for i in range(d):
        x = flat.view(flat.shape[0], -1, 2, 1 << i)
        x[:, :, 1] += x[:, :, 0]
    return a


def _mobius_(a, d):
    flat = a.view(-1, 1 << d)
    for i in range(d):
        x = flat.view(flat.shape[0], -1, 2, 1 << i)
        x[:, :, 1] -= x[:, :, 0]
    return a


def _scatter(out, masks, vals):
    out.index_add_(0, torch.from_numpy(masks).to(out.device),
                   torch.from_numpy(vals).to(out.device))


def _coeffs(rng, game, d):
    if game == "planted":
        return _planted_coeffs(rng, d, 200, 6)
    depth = 5
    p = _forest_params(rng, d, 100, depth)
    return _tree_coeffs(p, rng.random(d), rng.random(d), depth)


def _values(rng, games, d, dtype):
    """One row of 2^d values per entry of games, in the storage type. The
    factor gives the values full mantissas."""
    out = torch.empty((len(games), 1 << d), dtype=TORCH_DTYPE[dtype], device=DEV)
    step = max(1, (1 << 27) >> d)
    for i0 in range(0, len(games), step):
        part = games[i0:i0 + step]
        a = torch.zeros((len(part), 1 << d), dtype=torch.float64, device=DEV)
        for r, g in enumerate(part):
            _scatter(a[r], *_coeffs(rng, g, d))
        _zeta_(a, d)
        out[i0:i0 + step] = a.mul_(1.0 / 3.0)
    return out


def _sizes(case):
    """(d, l) of every instance of an operator case. The sizes of a ragged
    batch belong to the case, not to its inputs."""
    if case["kind"] == "ragged":
        rng = np.random.default_rng([case["n"], case["dlo"], case["dhi"]])
        ds = rng.integers(case["dlo"], case["dhi"] + 1, size=case["n"])
        ls = rng.integers(case["llo"], case["lhi"] + 1, size=case["n"])
        return [(int(d), int(l)) for d, l in zip(ds, ls)]
    return [(case["d"], case["l"])] * case.get("n", 1)


def _game_list(n):
    return ["tree" if i % 2 == 0 else "planted" for i in range(n)]


def _operator_values(case, seed):
    rng = np.random.default_rng([seed, 1])
    if case["kind"] == "single":
        return _values(rng, [case["game"]], case["d"], case["dtype"])[0]
    if case["kind"] == "batch":
        return _values(rng, _game_list(case["n"]), case["d"], case["dtype"]).view(-1)
    return torch.cat([_values(rng, [g], d, case["dtype"])[0]
                      for g, (d, _) in zip(_game_list(case["n"]), _sizes(case))])


def _forest_inputs(case, seed):
    rng = np.random.default_rng([seed, 2])
    p = _forest_params(rng, case["d"], case["trees"], case["depth"])
    x = torch.from_numpy(rng.random(case["d"])).to(DEV)
    bg = torch.from_numpy(rng.random((case["n_bg"], case["d"]))).to(DEV)
    return p, x, bg


def _make_forest(p, d, n_bg):
    """Node arrays of full binary trees: heap order inside a tree."""
    trees, inner = p["feat"].shape
    n = 2 * inner + 1
    feature = np.full((trees, n), -1, dtype=np.int32)
    feature[:, :inner] = p["feat"]
    thr = np.zeros((trees, n))
    thr[:, :inner] = p["thr"]
    value = np.zeros((trees, n))
    value[:, inner:] = p["leaf"]
    base = (np.arange(trees) * n)[:, None]
    child = np.arange(n)[None, :]
    isin = child < inner
    left = np.where(isin, base + 2 * child + 1, 0)
    right = np.where(isin, base + 2 * child + 2, 0)
    return Forest(d, base[:, 0], feature.ravel(), thr.ravel(), left.ravel(), right.ravel(),
                  value.ravel(), max_bg=n_bg)


# -------------------------------------------------------------- prepare / run
def prepare(case, seed):
    kind = case["kind"]
    dt = TORCH_DTYPE[case["dtype"]]
    if kind == "single":
        plan = Plan(case["d"], case["l"], dtype=case["dtype"], precision=case["precision"],
                    index=case["index"])
        return {"kind": kind, "plan": plan, "v": _operator_values(case, seed),
                "out": torch.empty(plan.M, dtype=dt, device=DEV)}
    if kind in ("batch", "ragged"):
        sizes = _sizes(case)
        plan = BatchPlan([d for d, _ in sizes], [l for _, l in sizes], dtype=case["dtype"],
                         precision=case["precision"], index=case["index"])
        return {"kind": kind, "plan": plan, "v": _operator_values(case, seed),
                "out": torch.empty(plan.out_offset[-1], dtype=dt, device=DEV)}
    if kind == "mobius":
        rng = np.random.default_rng([seed, 1])
        v = _values(rng, ["planted"], case["d"], case["dtype"])[0]
        return {"kind": kind, "plan": Plan(case["d"], 1, dtype=case["dtype"]), "v": v,
                "out": torch.empty_like(v)}
    p, x, bg = _forest_inputs(case, seed)
    d = case["d"]
    state = {"kind": kind, "forest": _make_forest(p, d, case["n_bg"]), "x": x, "bg": bg,
             "dtype": case["dtype"], "method": case.get("method", "mobius"),
             "v": torch.empty(1 << d, dtype=dt, device=DEV)}
    state["work"] = state["v"]
    if case["dtype"] == "f32":
        state["work"] = torch.empty(1 << d, dtype=torch.float64, device=DEV)
    if kind == "forest_fsi":
        state["plan"] = Plan(d, case["l"], dtype=case["dtype"])
        state["out"] = torch.empty(state["plan"].M, dtype=dt, device=DEV)
    return state


def run(state):
    kind = state["kind"]
    if kind in ("single", "batch", "ragged"):
        return state["plan"].apply(state["v"], out=state["out"])
    if kind == "mobius":
        state["out"].copy_(state["v"])
        return state["plan"].mobius(state["out"])
    v = state["forest"].values(state["x"], state["bg"], dtype=state["dtype"], out=state["v"],
                               method=state["method"], work=state["work"])
    if kind == "forest":
        return v
    return v, state["plan"].apply(v, out=state["out"])


# ----------------------------------------------------------------------- work
def _operator_work(d, l, item):
    """Values read and scores written once; a butterfly of d / 2 subtractions
    per value and the additions of the counter sweep (a site merges the two
    predecessors of every state that has both)."""
    outs = sum(math.comb(d, s) for s in range(l + 1))
    adds = sum((1 << (d - k)) * sum(math.comb(k - 1, s) * (k - 1 - s)
                                    for s in range(min(l, k - 1) + 1)) for k in range(1, d + 1))
    return item * ((1 << d) + outs), d * (1 << (d - 1)) + adds


def work(case):
    item = 4 if case["dtype"] == "f32" else 8
    kind = case["kind"]
    if kind in ("single", "batch", "ragged"):
        each = [_operator_work(d, l, item) for d, l in _sizes(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    d = case["d"]
    if kind == "mobius":
        return {"bytes": 2 * item << d, "flops": d << (d - 1)}
    nodes = case["trees"] * ((2 << case["depth"]) - 1)
    read = nodes * 28 + 8 * d * (1 + case["n_bg"])
    # one addition per coalition, tree and background on the walk; the subset
    # sums and one addition per reachable path on the Moebius route
    flops = (case["trees"] * case["n_bg"]) << d
    if kind == "forest_fsi" or case["method"] == "mobius":
        flops = (d << (d - 1)) + case["trees"] * case["n_bg"] * (1 << case["depth"])
    out = {"bytes": read + (item << d), "flops": flops}
    if kind == "forest_fsi":
        b, f = _operator_work(d, case["l"], item)
        out = {"bytes": out["bytes"] + b, "flops": out["flops"] + f}
    return out


# ---------------------------------------------------------------------- exact
def _bernoulli(n):
    b = []
    for m in range(n + 1):
        b.append(Fraction(1) if m == 0 else
                 -sum(math.comb(m + 1, i) * b[i] for i in range(m)) / Fraction(m + 1))
    return b


def _weight(s, t, l, index):
    if index == "stii":
        if s < l:
            return Fraction(int(t == s))
        return Fraction(1, math.comb(t, l))
    if index == "sii":
        return Fraction(1, t - s + 1)
    if index == "bii":
        return Fraction(1, 1 << (t - s))
    if index == "ksii":
        if s == 0:
            return Fraction(int(t == 0))
        n = t - s
        bern = _bernoulli(min(l - s, n))
        return sum((bern[j] * math.comb(n, j) / Fraction(n - j + 1) for j in range(len(bern))),
                   Fraction(0))
    if t == s:
        return Fraction(1)
    if t <= l or s == 0:
        return Fraction(0)
    w = Fraction(s * math.comb(l, s) * math.comb(t - 1, l),
                 (l + s) * math.comb(t + l - 1, l + s))
    return -w if (l - s) % 2 else w


def _popcount(d):
    p = torch.zeros(1, dtype=torch.int64, device=DEV)
    for _ in range(d):
        p = torch.cat([p, p + 1])
    return p


def _scores(v, d, l, index):
    """Scores of every row of v (rows, 2^d) in FP64: Moebius transform, then
    weighted superset sums per output size."""
    a = _mobius_(v.double().clone(), d)
    pop = _popcount(d)
    cols = []
    for s in range(l + 1):
        w = torch.tensor([float(_weight(s, t, l, index)) if t >= s else 0.0
                          for t in range(d + 1)], dtype=torch.float64, device=DEV)
        z = a * w[pop]
        for i in range(d):
            x = z.view(z.shape[0], -1, 2, 1 << i)
            x[:, :, 0] += x[:, :, 1]
        cols.append(z[:, torch.nonzero(pop == s).view(-1)])
    return torch.cat(cols, dim=1)


def _forest_exact(p, x, bg, d):
    trees, inner = p["feat"].shape
    depth = inner.bit_length()
    S = torch.arange(1 << d, device=DEV)
    feat = torch.from_numpy(p["feat"]).to(DEV)
    thr = torch.from_numpy(p["thr"]).to(DEV)
    leaf = torch.from_numpy(p["leaf"]).to(DEV)
    v = torch.zeros(1 << d, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 25) >> d)
    for b in range(bg.shape[0]):
        gx, gb = x[feat] >= thr, bg[b][feat] >= thr
        for t0 in range(0, trees, step):
            ft, xt, bt = feat[t0:t0 + step], gx[t0:t0 + step], gb[t0:t0 + step]
            node = torch.zeros((ft.shape[0], 1 << d), dtype=torch.int64, device=DEV)
            for _ in range(depth):
                inside = ((S[None, :] >> ft.gather(1, node)) & 1).bool()
                go = torch.where(inside, xt.gather(1, node), bt.gather(1, node))
                node = 2 * node + 1 + go
            v += leaf[t0:t0 + step].gather(1, node - inner).sum(dim=0)
    return v / bg.shape[0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "single":
        return _scores(_operator_values(case, seed).view(1, -1), case["d"], case["l"],
                       case["index"])[0]
    if kind == "batch":
        v = _operator_values(case, seed).view(case["n"], -1)
        step = max(1, (1 << 27) >> case["d"])
        return torch.cat([_scores(v[i:i + step], case["d"], case["l"], case["index"]).view(-1)
                          for i in range(0, case["n"], step)])
    if kind == "ragged":
        v = _operator_values(case, seed)
        out, at = [], 0
        for d, l in _sizes(case):
            out.append(_scores(v[at:at + (1 << d)].view(1, -1), d, l, case["index"])[0])
            at += 1 << d
        return torch.cat(out)
    if kind == "mobius":
        rng = np.random.default_rng([seed, 1])
        v = _values(rng, ["planted"], case["d"], case["dtype"])[0]
        return _mobius_(v.double(), case["d"])
    p, x, bg = _forest_inputs(case, seed)
    d = case["d"]
    v = _forest_exact(p, x, bg, d)
    if kind == "forest":
        return v
    return v, _scores(v.view(1, -1), d, case["l"], "fsi")[0]
