"""Performance cases of the symbolic-regression path, through the calls that
a program makes (paper_2602_06986_amd.Context): screening of candidate
expressions, exhaustive L0, branch and bound, annealing, OMP, and the whole
batched SISSO loop.

listed() holds twelve named cases, draw() others of the same ranges;
prepare() makes the inputs on the GPU, run() is one pass, work() what a pass
cannot do without, and exact() the results in 64 bits by plain torch and
numpy.  One library context serves the whole process, as it does in a
program that fits one dataset after another."""
import math

import numpy as np
import torch

import paper_2602_06986_amd as dm

UNARY = ("exp", "log", "sqrt", "sq", "inv")
BINARY = ("add", "sub", "mul", "div", "rdiv")
# base-unit exponents (length, mass, time) of a 16-feature dataset; other
# feature counts stretch the list
UNITS16 = np.array([[0, 0, 0]] * 4 + [[1, 0, 0]] * 3 + [[0, 1, 0]] * 3 + [[0, 0, 1]] * 3 + [[1, 0, -1]] * 2 +
                   [[2, 1, -2]], dtype=np.int32)


def listed():
    return [
        # a first look at a small table: one rung of all operators, top 20; latency
        {"name": "screen_first_look", "kind": "screen", "p": 6, "n": 100, "rung": 1, "T": 1, "units": False,
         "mode": "per_target", "precision": "fp64", "k": 20},
        # many responses measured on one small table, each with its own list
        {"name": "screen_16_targets", "kind": "screen", "p": 6, "n": 100, "rung": 2, "T": 16, "units": False,
         "mode": "per_target", "precision": "fp64", "k": 20},
        # the ordinary screen: 16 features with physical units, 500 samples, rung 2
        {"name": "screen_units16", "kind": "screen", "p": 16, "n": 500, "rung": 2, "T": 1, "units": True,
         "mode": "per_target", "precision": "fp64", "k": 500},
        # a wide dimensionless table with a ragged sample count, against 8 residuals
        {"name": "screen_dense20", "kind": "screen", "p": 20, "n": 1999, "rung": 2, "T": 8, "units": False,
         "mode": "max", "precision": "fp64", "k": 200},
        # the largest search: 24 features, rung 3, 8 residuals, precision form
        {"name": "screen_rung3_bf16", "kind": "screen", "p": 24, "n": 2000, "rung": 3, "T": 8, "units": True,
         "mode": "max", "precision": "bf16", "k": 1000},
        # a smaller rung-3 search wholly in FP64, first dimension
        {"name": "screen_rung3_fp64", "kind": "screen", "p": 15, "n": 777, "rung": 3, "T": 1, "units": True,
         "mode": "per_target", "precision": "fp64", "k": 300},
        # second dimension of a large loop: all pairs of 2000 rows, 8 models kept for their residuals
        {"name": "l0_pairs", "kind": "l0", "S": 2000, "n": 2000, "D": 2, "m": 8},
        # third dimension of an ordinary loop: all triples of 1500 rows
        {"name": "l0_triples", "kind": "l0", "S": 1500, "n": 500, "D": 3, "m": 1},
        # greedy extension over a large union subspace
        {"name": "omp", "kind": "omp", "S": 3000, "n": 2000, "D": 6},
        # stochastic search where exhaustive L0 is out of reach
        {"name": "anneal", "kind": "anneal", "S": 3000, "n": 2000, "D": 6, "chains": 16384, "steps": 2000},
        # exact search beyond three terms
        {"name": "bnb", "kind": "bnb", "S": 400, "n": 1600, "D": 5, "m": 1},
        # the whole loop over a batch of uneven datasets, then OMP; replays of the captured loop
        {"name": "loop_batch8", "kind": "loop", "datasets": 8, "p_lo": 6, "p_hi": 20, "n_lo": 50, "n_hi": 2000,
         "rung": 2, "k": 200, "D": 3, "m": 1, "omp": 5},
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of lo..hi."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["screen", "screen", "screen", "screen", "rung3", "rung3", "l0", "l0", "l0", "omp", "anneal",
                       "bnb", "loop"])
    if kind == "screen":
        rung = rng.choice([1, 2, 2, 2])
        T = rng.choice([1, 1, 2, 3, 5, 8, 16])
        return {"kind": "screen", "p": _log(rng, 4, 24 if T < 16 else 16), "n": _log(rng, 40, 2000), "rung": rung,
                "T": T, "units": rng.random() < 0.5, "mode": "max" if T > 1 and rng.random() < 0.6 else "per_target",
                "precision": rng.choice(["fp64", "fp64", "bf16", "fp16"]), "k": _log(rng, 5, 30 if rung == 1 else 500)}
    if kind == "rung3":
        T = rng.choice([1, 2, 4, 8])
        return {"kind": "screen", "p": rng.randint(6, 18), "n": _log(rng, 60, 1500), "rung": 3, "T": T, "units": True,
                "mode": "max" if T > 1 else "per_target", "precision": rng.choice(["bf16", "bf16", "fp64"]),
                "k": _log(rng, 20, 800)}
    if kind == "l0":
        D = rng.randint(1, 3)
        return {"kind": "l0", "S": _log(rng, 20, 1500 if D == 3 else 3000), "n": _log(rng, 50, 2000), "D": D,
                "m": rng.choice([1, 1, 2, 8, 16])}
    if kind == "omp":
        return {"kind": "omp", "S": _log(rng, 50, 3000), "n": _log(rng, 50, 2000), "D": rng.randint(2, 8)}
    if kind == "anneal":
        return {"kind": "anneal", "S": _log(rng, 100, 3000), "n": _log(rng, 50, 2000), "D": rng.randint(2, 6),
                "chains": _log(rng, 512, 16384), "steps": _log(rng, 200, 2000)}
    if kind == "bnb":
        return {"kind": "bnb", "S": _log(rng, 32, 256), "n": _log(rng, 100, 1500), "D": rng.choice([3, 4, 5]),
                "m": rng.choice([1, 1, 4])}
    lo = _log(rng, 40, 300)
    return {"kind": "loop", "datasets": rng.randint(1, 6), "p_lo": rng.randint(4, 6), "p_hi": rng.randint(7, 16),
            "n_lo": lo, "n_hi": _log(rng, lo + 10, 1500), "rung": 2, "k": _log(rng, 20, 150), "D": rng.randint(2, 3),
            "m": rng.choice([1, 1, 4]), "omp": 5}


# ------------------------------------------------------------------ inputs
def _dataset(rng, p, n, units):
    """p primary features [p][n], their unit exponents or None, and a target
    of five products of features with 1 % noise."""
    X = rng.lognormal(0.0, 0.5, size=(p, n)) if units else rng.uniform(0.5, 2.0, size=(p, n))
    y = np.full(n, 0.5)
    terms = []
    for c in (2.0, -1.3, 0.8, 0.3, -0.2):
        cols = rng.choice(p, size=3, replace=False)
        t = X[cols[0]] * X[cols[1]] / X[cols[2]]
        terms.append(t)
        y = y + c * (t - t.mean()) / t.std()
    y = y + rng.normal(0.0, 0.01 * y.std(), size=n)
    U = UNITS16[np.arange(p) * 16 // p] if units else None
    return X, y, U, terms


def _screen_host(case, seed):
    rng = np.random.default_rng(1000003 * seed + 17)
    X, y, U, terms = _dataset(rng, case["p"], case["n"], case["units"])
    Y = [y]
    for t in range(1, case["T"]):
        if case["mode"] == "max":
            # residuals of several good one-term models: alike, as those of a loop's next dimension are
            f = terms[0] * X[t % case["p"]] ** (0.02 * t)
            f = f - f.mean()
            Y.append(y - y.mean() - f * (f @ y) / (f @ f))
        else:
            Y.append(rng.permutation([1.5, -1.0, 0.6, 0.3, 0.1]) @ np.array(terms) + rng.normal(0.0, 0.01, case["n"]))
    if case["mode"] == "max":
        f = terms[0] - terms[0].mean()
        Y[0] = y - y.mean() - f * (f @ y) / (f @ f)
    return X, np.array(Y), U


def _subspace(case, seed, dev):
    """Rows as a screening leaves them: products of powers of a few latent
    features, most of them variants of the target's terms; IDs ascending."""
    rng = np.random.default_rng(1000003 * seed + 29)
    S, n, D, p = case["S"], case["n"], case["D"], 24
    Z = rng.normal(0.0, 0.5, size=(p, n))
    base = np.zeros((D, p))
    for d in range(D):
        base[d, rng.choice(p, size=2, replace=False)] = rng.choice([-1, 1, 2], size=2)
    seen = {tuple(b) for b in base}
    W = [b for b in base]
    while len(W) < S:
        w = base[rng.integers(D)].copy() if rng.random() < 0.7 else np.zeros(p)
        w[rng.choice(p, size=int(rng.integers(1, 4)), replace=False)] = rng.choice([-2, -1, 1, 2])
        if w.any() and tuple(w) not in seen and tuple(-w) not in seen:
            seen.add(tuple(w))
            W.append(w)
    at = rng.permutation(S)
    W = np.array(W)[at]
    F = torch.exp(torch.as_tensor(W, device=dev) @ torch.as_tensor(Z, device=dev))
    rows = np.argsort(at)[:D]
    G = F[torch.as_tensor(rows, device=dev)]
    G = (G - G.mean(1, keepdim=True)) / G.std(1, keepdim=True)
    c = torch.as_tensor(rng.uniform(0.5, 2.0, D) * rng.choice([-1.0, 1.0], D), device=dev)
    y = 0.5 + c @ G
    y = y + 0.1 * y.std() * torch.as_tensor(rng.normal(size=n), device=dev)
    ids = np.sort(rng.choice(700_000_000, size=S, replace=False)).astype(np.int64)
    return F.contiguous(), torch.as_tensor(ids, device=dev), y.contiguous()


def _loop_host(case, seed):
    rng = np.random.default_rng(1000003 * seed + 41)
    sizes = np.random.default_rng(case["datasets"] * 7919 + case["n_hi"])
    out = []
    for b in range(case["datasets"]):
        n = int(sizes.integers(case["n_lo"], case["n_hi"] + 1))
        p = int(sizes.integers(case["p_lo"], case["p_hi"] + 1))
        X, y, _, _ = _dataset(rng, p, n, False)
        out.append((X, y))
    return out


def _params(case):
    if case["kind"] == "loop":
        return dm.params(rung=case["rung"], k=case["k"])
    more = {"rung_ops": (None, None, None, BINARY), "rung_pool": (None, None, None, 0)} if case["rung"] == 3 else {}
    return dm.params(rung=case["rung"], k=case["k"],
                     score_mode=dm.SCORE_MAX if case["mode"] == "max" else dm.SCORE_PER_TARGET,
                     precision={"fp64": dm.FP64, "bf16": dm.BF16_GUARD, "fp16": dm.FP16_GUARD}[case["precision"]], **more)


_ctx = []


def _context():
    if not _ctx:
        _ctx.append(dm.Context(0))
    return _ctx[0]


def prepare(case, seed):
    dev = torch.device("cuda:0")
    s = {"case": case, "ctx": _context(), "kind": case["kind"]}
    if case["kind"] == "screen":
        X, Y, U = _screen_host(case, seed)
        s.update(X=torch.as_tensor(X, device=dev), Y=torch.as_tensor(Y, device=dev), units=U, prm=_params(case))
    elif case["kind"] == "loop":
        data = _loop_host(case, seed)
        s.update(Xs=[torch.as_tensor(X, device=dev) for X, _ in data],
                 ys=[torch.as_tensor(y, device=dev) for _, y in data], prm=_params(case))
    else:
        s["F"], s["ids"], s["y"] = _subspace(case, seed, dev)
    return s


def run(s):
    c, ctx = s["case"], s["ctx"]
    if s["kind"] == "screen":
        ids, scores, values, _ = ctx.generate_screen(s["X"], s["Y"], s["prm"], units=s["units"])
        return {"ids": ids, "scores": scores, "values": values}
    if s["kind"] == "loop":
        ids, scores, sub, rmse, coef, _, omp = ctx.sisso_batch_graph(s["Xs"], s["ys"], s["prm"], c["D"], m=c["m"],
                                                                     omp_D=c["omp"])
        return {"ids": ids, "scores": scores, "subsets": sub, "rmse": rmse, "coef": coef, "omp": omp}
    if s["kind"] == "l0":
        sub, rmse, coef, resid, _ = ctx.l0_fit(s["F"], s["ids"], s["y"], c["D"], c["m"])
    elif s["kind"] == "bnb":
        sub, rmse, coef, resid, _ = ctx.l0_bnb(s["F"], s["ids"], s["y"], c["D"], c["m"])
    elif s["kind"] == "omp":
        sub, coef, rmse, resid = ctx.omp(s["F"], s["ids"], s["y"], c["D"])
    else:
        sub, rmse, coef, energy, _, _, resid = ctx.anneal(s["F"], s["ids"], s["y"], c["D"], chains=c["chains"],
                                                          steps=c["steps"], seed=7, resid=True)
        return {"subsets": sub, "rmse": rmse, "coef": coef, "energy": energy, "resid": resid}
    return {"subsets": sub, "rmse": rmse, "coef": coef, "resid": resid}


# -------------------------------------------------- the search space, plainly
class _Space:
    """Rungs 0..2 of the search space: for every unit-legal feature its rung,
    ID, operator and operands; units as one integer key (0: dimensionless)."""

    def __init__(self, p, U, rung):
        # exponents scaled by 8 so that square roots stay whole, packed into one integer
        key = np.zeros(p, np.int64) if U is None else (U.astype(np.int64) * 8) @ np.array([1, 1 << 16, 1 << 32])
        self.raw = p
        self.id, self.op, self.i, self.j = np.arange(p), np.full(p, -1), np.full(p, -1), np.full(p, -1)
        self.key, self.rung = key, np.zeros(p, np.int64)
        for r in range(1, min(rung, 2) + 1):
            self._grow(r)

    def _grow(self, r):
        # positions of rung r - 1's raw features, and which of them are legal (compact index or -1)
        at = np.full(self.raw, -1)
        at[self.id] = np.arange(len(self.id))
        lo = 0 if r == 1 else self.first
        new = []
        base = self.raw
        for o, name in enumerate(UNARY):
            c = at[lo:self.raw]
            ok = c >= 0
            k = self.key[np.maximum(c, 0)]
            if name in ("exp", "log"):
                ok = ok & (k == 0)
            new.append((base + np.flatnonzero(ok), o, c[ok], np.full(int(ok.sum()), -1),
                        {"exp": k, "log": k, "sqrt": k // 2, "sq": 2 * k, "inv": -k}[name][ok]))
            base += self.raw - lo
        jj = np.arange(lo, self.raw)
        J = np.repeat(jj, jj)
        I = np.arange(len(J)) - np.repeat(np.cumsum(jj) - jj, jj)
        ci, cj = at[I], at[J]
        legal = (ci >= 0) & (cj >= 0)
        ki, kj = self.key[np.maximum(ci, 0)], self.key[np.maximum(cj, 0)]
        for o, name in enumerate(BINARY):
            ok = legal & (ki == kj) if name in ("add", "sub") else legal
            k = {"add": ki, "sub": ki, "mul": ki + kj, "div": ki - kj, "rdiv": kj - ki}[name]
            new.append((base + np.flatnonzero(ok), 5 + o, ci[ok], cj[ok], k[ok]))
            base += len(J)
        self.first, self.raw = self.raw, base
        self.id = np.concatenate([self.id] + [a[0] for a in new])
        self.op = np.concatenate([self.op] + [np.full(len(a[0]), a[1]) for a in new])
        self.i = np.concatenate([self.i] + [a[2] for a in new])
        self.j = np.concatenate([self.j] + [a[3] for a in new])
        self.key = np.concatenate([self.key] + [a[4] for a in new])
        self.rung = np.concatenate([self.rung] + [np.full(len(a[0]), r) for a in new])

    def count3(self, p):
        """Unit-legal candidates with the operator-limited rung 3 (binary
        operators, partner a primary) added."""
        g = self.rung == 2
        n = 3 * p * int(g.sum())
        for k in self.key[:p]:
            n += 2 * int((g & (self.key == k)).sum())
        return len(self.id) + n


def work(case):
    c, k = case, case["kind"]
    if k == "screen":
        sp = _Space(c["p"], UNITS16[np.arange(c["p"]) * 16 // c["p"]] if c["units"] else None, c["rung"])
        cand = sp.count3(c["p"]) if c["rung"] == 3 else len(sp.id)
        lists = 1 if c["mode"] == "max" else c["T"]
        # an operator, the mean, the variance, and a dot product per target for each sample of each candidate
        return {"bytes": 8 * ((c["p"] + c["T"]) * c["n"] + lists * c["k"] * (c["n"] + 2)),
                "flops": (4 + 2 * c["T"]) * c["n"] * cand}
    if k == "loop":
        by = fl = 0
        sizes = np.random.default_rng(c["datasets"] * 7919 + c["n_hi"])
        for _ in range(c["datasets"]):
            n = int(sizes.integers(c["n_lo"], c["n_hi"] + 1))
            p = int(sizes.integers(c["p_lo"], c["p_hi"] + 1))
            cand = len(_Space(p, None, c["rung"]).id)
            by += 8 * ((p + 1) * n + 2 * c["D"] * c["k"])
            for d in range(1, c["D"] + 1):
                S = d * c["k"]
                fl += (4 + 2 * (1 if d == 1 else c["m"])) * n * cand + n * S * S + 12 * math.comb(S, d)
        return {"bytes": by, "flops": fl}
    S, n, D = c["S"], c["n"], c["D"]
    by = 8 * (S * n + S + n) + 8 * n * c.get("m", 1)
    if k == "l0":
        return {"bytes": by, "flops": n * S * S + 12 * math.comb(S, D)}
    if k == "omp":
        return {"bytes": by, "flops": 2 * n * S * D}
    if k == "anneal":  # the correlation matrix and, per proposal, one row of a Cholesky factor at least
        return {"bytes": by, "flops": n * S * S + c["chains"] * c["steps"] * D * D}
    return {"bytes": by, "flops": n * S * S + 12 * math.comb(S, 2)}


# --------------------------------------------------------------- 64-bit results
def _apply(op, a, b):
    return (lambda: torch.exp(a), lambda: torch.log(a), lambda: torch.sqrt(a), lambda: a * a, lambda: 1.0 / a,
            lambda: a + b, lambda: a - b, lambda: a * b, lambda: a / b, lambda: b / a)[op]()


def _score(f, ok, Yc, ab):
    """|Pearson r| [rows][T] of the rows of f (-1 where a row is invalid),
    and which rows are valid; ab: sum of the operands' squares for a sum or
    difference, else None."""
    n = f.shape[1]
    sf = (f * f).sum(1)
    d = f - f.mean(1, keepdim=True)
    ss = (d * d).sum(1)
    ok = ok & torch.isfinite(sf) & torch.isfinite(ss) & (torch.sqrt(ss / n) > 1e-8 * torch.sqrt(sf / n))
    if ab is not None:
        ok = ok & (sf > 1e-20 * ab)
    r = (d @ Yc).abs() / torch.sqrt(ss)[:, None]
    return torch.where(ok[:, None], r, torch.full_like(r, -1.0)), ok


class _Screen64:
    """Every candidate of one dataset scored in 64 bits, and the exact
    selection: order by (-score, ID), near-tie duplicates merged under their
    smallest ID, groups holding an excluded ID dropped."""

    def __init__(self, X, U, rung, dev):
        self.dev, self.rung, self.p = dev, rung, X.shape[0]
        self.sp = _Space(self.p, U, rung)
        self.n = X.shape[1]
        self.keep = int((self.sp.rung < max(rung, 1)).sum())     # features whose values are held as operands
        self.V = torch.empty((self.keep, self.n), dtype=torch.float64, device=dev)
        self.V[:self.p] = torch.as_tensor(X, device=dev)
        self.ok = torch.zeros(self.keep, dtype=torch.bool, device=dev)
        zero = torch.zeros((self.n, 1), dtype=torch.float64, device=dev)
        self.ok[:self.p] = _score(self.V[:self.p], torch.ones(self.p, dtype=torch.bool, device=dev), zero, None)[1]
        for lo, hi, f, ab, ok in self._rows(self.p, self.keep):
            self.V[lo:hi] = f
            self.ok[lo:hi] = _score(f, ok, zero, ab)[1]

    def _rows(self, lo, end):
        """Values of the legal features lo..end in chunks of one operator."""
        step = max(1, (1 << 27) // self.n)
        while lo < end:
            op = int(self.sp.op[lo])
            hi = lo + 1
            same = np.flatnonzero(self.sp.op[lo:min(end, lo + step)] != op)
            hi = lo + (int(same[0]) if len(same) else min(step, end - lo))
            f, ab, ok = self.values(op, self.sp.i[lo:hi], self.sp.j[lo:hi])
            yield lo, hi, f, ab, ok
            lo = hi

    def values(self, op, i, j):
        """Values of one operator's rows, the sum of their operands' squares
        where they are sums or differences, and whether the operands are valid."""
        i = torch.as_tensor(i, device=self.dev)
        a, ok, b, ab = self.V[i], self.ok[i], None, None
        if op >= 5:
            j = torch.as_tensor(j, device=self.dev)
            b, ok = self.V[j], ok & self.ok[j]
            ab = (a * a).sum(1) + (b * b).sum(1) if op < 7 else None
        return _apply(op, a, b), ab, ok

    def _candidates(self):
        """(IDs, f, sum of operand squares, valid) of every legal candidate."""
        yield torch.arange(self.p, device=self.dev), self.V[:self.p], None, self.ok[:self.p]
        for lo, hi, f, ab, ok in self._rows(self.p, len(self.sp.id) if self.rung < 3 else self.keep):
            yield torch.as_tensor(self.sp.id[lo:hi], device=self.dev), f, ab, ok
        if self.rung < 3:
            return
        sp, p = self.sp, self.p
        g = np.flatnonzero(sp.rung == 2)
        pairs = (sp.raw - sp.first) * p
        step = max(1, (1 << 28) // self.n)
        for x in range(p):
            xv = self.V[x]
            for at in range(0, len(g), step):
                j = g[at:at + step]
                b, okj = self.V[j[0]:j[-1] + 1], self.ok[j[0]:j[-1] + 1] & self.ok[x]
                idj = torch.as_tensor(sp.raw + (sp.id[j] - sp.first) * p + x, device=self.dev)
                for o in (7, 8, 9):
                    yield idj + (o - 5) * pairs, _apply(o, xv, b), None, okj
                same = np.flatnonzero(sp.key[j] == sp.key[x])
                if len(same):
                    t = torch.as_tensor(same, device=self.dev)
                    bs = b[t]
                    ab = (xv * xv).sum() + (bs * bs).sum(1)
                    for o in (5, 6):
                        yield idj[t] + (o - 5) * pairs, _apply(o, xv, bs), ab, okj[t]

    def row(self, cid):
        """The values of candidate cid."""
        sp, p = self.sp, self.p
        if cid >= sp.raw and self.rung == 3:
            pairs = (sp.raw - sp.first) * p
            o, rest = divmod(cid - sp.raw, pairs)
            return _apply(5 + o, self.V[rest % p], self.V[np.searchsorted(sp.id, sp.first + rest // p)])
        at = int(np.searchsorted(sp.id, cid))
        if at < self.keep:
            return self.V[at]
        return self.values(int(sp.op[at]), sp.i[at:at + 1], sp.j[at:at + 1])[0][0]

    def select(self, Y, k, use_max, exclude=()):
        """Per list (scores [k], IDs [k]), NaN and -1 past the selected ones."""
        Yc = torch.as_tensor(Y, device=self.dev)
        Yc = Yc - Yc.mean(1, keepdim=True)
        Yc = (Yc / Yc.norm(dim=1, keepdim=True)).T.contiguous()
        lists = 1 if use_max else Yc.shape[1]
        most = 16 * k + 4 * len(exclude) + 2000
        best = [(torch.empty(0, dtype=torch.float64, device=self.dev), torch.empty(0, dtype=torch.int64, device=self.dev))
                for _ in range(lists)]
        for ids, f, ab, ok in self._candidates():
            sc = _score(f, ok, Yc, ab)[0]
            sc = sc.max(1, keepdim=True)[0] if use_max else sc
            for q in range(lists):
                v = sc[:, q]
                if len(best[q][0]) >= most:
                    at = v > best[q][0].min()
                    v, w = v[at], ids[at]
                else:
                    w = ids
                if v.numel():
                    v, w = torch.cat([best[q][0], v]), torch.cat([best[q][1], w])
                    top = torch.topk(v, min(most, v.numel()))[1]
                    best[q] = (v[top], w[top])
        return [self._groups(v.cpu().numpy(), w.cpu().numpy(), k, set(int(e) for e in exclude)) for v, w in best]

    def _groups(self, sc, ids, k, exclude):
        at = np.lexsort((ids, -sc))
        sc, ids = sc[at], ids[at]
        sc, ids = sc[sc > 0], ids[sc > 0]
        heads = []                                  # [score of the smallest ID, smallest ID, blocked]
        lo = 0
        while lo < len(sc) and sum(not h[2] for h in heads) < k:
            hi = lo + 1
            while hi < len(sc) and sc[hi] >= sc[hi - 1] * (1 - 1e-9):
                hi += 1
            R = torch.stack([self.row(int(v)) for v in ids[lo:hi]]) if hi - lo > 1 else None
            if R is not None:
                R = R - R.mean(1, keepdim=True)
                R = R / R.norm(dim=1, keepdim=True)
            free = np.ones(hi - lo, bool)
            for e in range(hi - lo):
                if not free[e]:
                    continue
                member = np.zeros(hi - lo, bool)
                member[e] = True
                if R is not None:
                    same = (R[e:] @ R[e]).abs().cpu().numpy() >= 1 - 1e-9
                    member[e:] |= same & free[e:] & (sc[lo + e:hi] >= sc[lo + e] * (1 - 1e-9))
                free[member] = False
                got = np.flatnonzero(member) + lo
                s = got[np.argmin(ids[got])]
                heads.append([sc[s], ids[s], any(int(v) in exclude for v in ids[got])])
            lo = hi
        heads = sorted([h for h in heads if not h[2]][:k], key=lambda h: (-h[0], h[1]))
        s, i = np.full(k, np.nan), np.full(k, -1, np.int64)
        s[:len(heads)], i[:len(heads)] = [h[0] for h in heads], [h[1] for h in heads]
        return s, i


def _fit(F, y, rows):
    """Least squares of y on [1, rows of F]: RSS, coefficients, residual."""
    A = np.concatenate([np.ones((len(y), 1)), F[list(rows)].T], axis=1)
    scale = np.linalg.norm(A, axis=0)
    c = np.linalg.lstsq(A / scale, y, rcond=None)[0] / scale
    r = y - A @ c
    return float(r @ r), c, r


def _l0(F, ids, y, D, m):
    """The m best D-subsets: scanned through the correlation matrix, the best
    of the scan refitted."""
    dev = F.device
    Z = F - F.mean(1, keepdim=True)
    Z = Z / Z.norm(dim=1, keepdim=True)
    yc = y - y.mean()
    yc = yc / yc.norm()
    S = F.shape[0]
    found = []                                      # (explained fraction, rows)
    want = m + 64

    def scan(G, c, first, base, lo):
        """Completes the prefix `first` (explained fraction base) from the
        rows lo.. of a system G, c in which it has been eliminated."""
        left = D - len(first)
        d = torch.diagonal(G).clone()
        good = d > 1e-10
        q = torch.where(good, c * c / torch.where(good, d, torch.ones_like(d)), torch.full_like(d, -9.0))
        if left == 1:
            v, at = torch.topk(q[lo:], min(want, S - lo))
            keep(base + v, [first + (int(a) + lo,) for a in at.cpu().numpy()])
        elif left == 2:
            b = slice(lo, S)
            g, db, qb, cb = G[b, b], d[b], q[b], c[b]
            t = g / torch.where(good[b], db, torch.ones_like(db))[:, None]
            den = db[None, :] - t * g
            e = cb[None, :] - t * cb[:, None]
            v = torch.where(den > 1e-10, qb[:, None] + e * e / den, torch.full_like(g, -9.0))
            v = torch.triu(v + 9.0, 1) - 9.0
            v, at = torch.topk(v.reshape(-1), min(want, v.numel()))
            at = at.cpu().numpy()
            keep(base + v, [first + (int(a) // (S - lo) + lo, int(a) % (S - lo) + lo) for a in at])
        else:
            dh = d.cpu().numpy()
            for a in range(lo, S - left + 1):
                if dh[a] > 1e-10:
                    u = G[a] / d[a]
                    scan(G - u[:, None] * G[a][None, :], c - u * c[a], first + (a,), base + q[a], a + 1)

    def keep(v, rows):
        v = v.cpu().numpy()
        worst = min(found)[0] if len(found) >= want else -1.0
        found.extend((float(x), r) for x, r in zip(v, rows) if x > worst and x > 0)
        if len(found) > want:
            found.sort(reverse=True)
            del found[want:]

    scan(Z @ Z.T, Z @ yc, (), torch.zeros((), dtype=torch.float64, device=dev), 0)
    Fh, yh = F.cpu().numpy(), y.cpu().numpy()
    fits = sorted((_fit(Fh, yh, r)[0], r) for _, r in found)[:m]
    return [(r,) + _fit(Fh, yh, r) for _, r in fits]


def _omp(F, y, D, start=()):
    Fh, yh = F.cpu().numpy(), y.cpu().numpy()
    Z = F - F.mean(1, keepdim=True)
    Z = Z / Z.norm(dim=1, keepdim=True)
    act = list(start)
    r = _fit(Fh, yh, act)[2] if act else yh - yh.mean()
    while len(act) < D:
        c = (Z @ torch.as_tensor(r, device=F.device)).abs()
        c[act] = -1.0
        act.append(int(c.argmax()))
        r = _fit(Fh, yh, act)[2]
    rss, coef, r = _fit(Fh, yh, act)
    return act, coef, math.sqrt(rss / len(yh)), r


def exact(case, seed):
    dev = torch.device("cuda:0")
    c = case
    if c["kind"] == "screen":
        X, Y, U = _screen_host(c, seed)
        s = _Screen64(X, U, c["rung"], dev)
        got = s.select(Y, c["k"], c["mode"] == "max")
        if any((i < 0).any() for _, i in got):
            return None
        return {"ids": None, "scores": np.array([v for v, _ in got]),
                "values": torch.stack([torch.stack([s.row(int(v)) for v in i]) for _, i in got])}
    if c["kind"] == "anneal":
        return None                                 # a seeded random walk
    if c["kind"] == "loop":
        return _loop64(c, seed, dev)
    F, ids, y = _subspace(c, seed, dev)
    if c["kind"] == "omp":
        act, coef, rmse, r = _omp(F, y, c["D"])
        return {"subsets": None, "coef": coef, "rmse": np.array([rmse]), "resid": r}
    if c["D"] > 3 and math.comb(c["S"], c["D"] - 2) > 33000:
        return None                                 # every subset takes too long here
    fits = _l0(F, ids, y, c["D"], c["m"])
    if len(fits) < c["m"]:
        return None
    return {"subsets": None, "rmse": np.array([math.sqrt(f[1] / c["n"]) for f in fits]),
            "coef": np.array([f[2] for f in fits]), "resid": np.array([f[3] for f in fits])}


def _loop64(c, seed, dev):
    nb, D, m, k = c["datasets"], c["D"], c["m"], c["k"]
    data = _loop_host(c, seed)
    if sum(len(_Space(X.shape[0], None, 2).id) * X.shape[1] for X, _ in data) * (D + 1) > 1.5e11 or c["omp"] <= D:
        return None
    scores = np.full((nb, D, k), np.nan)
    rmse, coef = np.full((nb, D, m), np.nan), np.full((nb, D, m, 4), np.nan)
    ocoef, ormse = np.full((nb, c["omp"] + 1), np.nan), np.full(nb, np.nan)
    for b, (X, yh) in enumerate(data):
        s = _Screen64(X, None, c["rung"], dev)
        y = torch.as_tensor(yh, device=dev)
        ids, F, Y = [], torch.empty((0, len(yh)), dtype=torch.float64, device=dev), yh[None, :]
        for d in range(1, D + 1):
            (sc, got), = s.select(Y, k, len(Y) > 1, ids)
            if (got < 0).any():
                return None
            scores[b, d - 1] = sc
            ids += [int(v) for v in got]
            F = torch.cat([F, torch.stack([s.row(int(v)) for v in got])])
            fits = _l0(F, ids, y, d, m)
            if len(fits) < m:
                return None
            Y = np.array([f[3] for f in fits])
            for q, f in enumerate(fits):
                rmse[b, d - 1, q] = math.sqrt(f[1] / len(yh))
                coef[b, d - 1, q, :d + 1] = f[2]
        _, ocoef[b], ormse[b], _ = _omp(F, y, c["omp"], fits[0][0])
    return {"ids": None, "scores": scores, "subsets": None, "rmse": rmse, "coef": coef, "omp": [None, ocoef, ormse]}
