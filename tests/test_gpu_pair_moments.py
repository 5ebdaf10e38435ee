"""Moments of the FP64 pair screen: scores as accurate as sums over centred
values give them, on columns of any spread about their mean, and only a
small share of the candidates left to the exact fix-up, also where one
column lies far from zero or columns are nearly multiples of one another."""
import numpy as np
import pytest

from tests.checks import check_selection

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _status(torch, D, c, Xd, Yd, q, cap):
    """Outcome of a call whose fix-up lists hold cap entries."""
    c.set_fixup_capacity(cap)
    got = c.generate_screen(Xd, Yd, q, device_stats=True)
    torch.cuda.synchronize()
    return D.decode_stats(got[3], D.ScreenStats)[0]["status"]


@pytest.mark.parametrize("spread", [0.3, 1e-2, 3e-4, 1e-6])
@pytest.mark.parametrize("p,n,T", [(8, 64, 1), (9, 129, 3), (7, 1001, 2)])
def test_score_error(spread, p, n, T):
    """Screening scores of the pool against its exact scores: at most the
    bound of the moments, 4 n u 64, and of values rounded before they are
    centred, 3 u rms / std (a pair's own std may be an eighth of its
    operands' at that conditioning)."""
    import torch
    import paper_2602_06986_amd as D
    rng = np.random.default_rng(100 * p + n)
    Z = np.clip(rng.normal(size=(p, n)), -3, 3)
    X = np.exp(rng.uniform(-3, 6, size=(p, 1))) * (1.0 + spread * Z)
    Y = np.array([Z[t] * Z[(t + 1) % p] + 0.3 * Z[(t + 2) % p] + 0.1 * rng.normal(size=n) for t in range(T)])
    # (rung 1: the pairs of the primaries themselves)
    q = D.params(rung=1, k=30, ops=("add", "sub", "mul", "div", "rdiv"), score_mode=D.SCORE_MAX)
    c = D.Context(0)
    try:
        ids, sc, _, st = c.generate_screen(torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda"), q)
    finally:
        c.close()
    assert int((ids >= 0).sum()) > 10
    assert st["max_lowprec_err"] <= 4 * n * U * 64 + 3 * U * 8 / spread, st["max_lowprec_err"]


@pytest.mark.parametrize("kind", ["plain", "pressure", "all_narrow", "multiples"])
@pytest.mark.parametrize("T,mode", [(1, "per_target"), (3, "max")])
def test_fixup_share(oracle_mod, kind, T, mode):
    """At most 1 in 64 candidates is listed for the exact fix-up: one column
    of a mean thousands of times its spread among others (its sums with every
    column of a smaller scale), all columns such.  Where columns are multiples
    of one another to 0.2 % (their quotients cancel), the vector form is
    taken: no more than it lists."""
    import torch
    import paper_2602_06986_amd as D
    O = oracle_mod
    p, n, k = (16 if kind == "pressure" else 10), 60, 15
    rng = np.random.default_rng(5)
    X = rng.lognormal(0.0, 0.5, size=(p, n))
    if kind == "pressure":
        X[0] = 101325.0 + 10.0 * rng.normal(size=n)
    elif kind == "all_narrow":
        X = 300.0 + 0.3 * rng.normal(size=(p, n))
    elif kind == "multiples":
        X = np.arange(1, p + 1)[:, None] * X[0] * (1.0 + 2e-3 * rng.normal(size=(p, n)))
    Z = (X - X.mean(1, keepdims=True)) / X.std(1, keepdims=True)
    Y = np.array([Z[t] + Z[t + 1] * Z[t + 2] + 0.1 * rng.normal(size=n) for t in range(T)])
    q = D.params(rung=2, k=k, score_mode=D.SCORE_MAX if mode == "max" else D.SCORE_PER_TARGET)
    sp = O.Space(p, 2, O.OPS)
    lists, _, nvalid = O.sis(sp, X, None, Y, k, (), mode)
    c = D.Context(0)
    try:
        Xd, Yd = torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda")
        ids, sc, _, st = c.generate_screen(Xd, Yd, q)
        assert st["n_scored"] == nvalid
        for t in range(len(lists)):
            check_selection(ids[t].cpu().numpy(), sc[t].cpu().numpy(), lists[t][0], lists[t][1])
        cap = nvalid // 64
        if kind == "multiples":
            qv = D.params(rung=2, k=k, score_mode=q.score_mode, tile_j=1)
            c.generate_screen(Xd, Yd, qv)
            lo, hi = 0, nvalid
            while hi - lo > 1:
                mid = (lo + hi) // 2
                lo, hi = (lo, mid) if _status(torch, D, c, Xd, Yd, qv, mid) == 0 else (mid, hi)
            cap = hi
        assert _status(torch, D, c, Xd, Yd, q, cap) == 0
    finally:
        c.close()


def test_batch_of_both_forms():
    """One call over datasets of which some take the matrix form and some
    the vector form equals the calls apart."""
    import torch
    import paper_2602_06986_amd as D
    rng = np.random.default_rng(3)
    Xs, Ys = [], []
    for b, (p, n) in enumerate([(8, 60), (7, 45), (11, 130), (9, 33)]):
        X = rng.lognormal(0.0, 0.5, size=(p, n))
        if b % 2:
            X = np.arange(1, p + 1)[:, None] * X[0] * (1.0 + 2e-3 * rng.normal(size=(p, n)))
        Xs.append(torch.as_tensor(X, device="cuda"))
        Ys.append(torch.as_tensor((X[0] * X[1] / X[2] + 0.1 * rng.normal(size=n))[None], device="cuda"))
    q = D.params(rung=2, k=15)
    c = D.Context(0)
    try:
        both = c.generate_screen_batch(Xs, Ys, q)
        for b in range(len(Xs)):
            ids, sc, vals, st = c.generate_screen(Xs[b], Ys[b], q)
            assert torch.equal(ids, both[b][0]) and torch.equal(sc, both[b][1]) and torch.equal(vals, both[b][2])
            assert st["n_scored"] == both[b][3]["n_scored"]
    finally:
        c.close()
