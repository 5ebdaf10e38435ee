"""The precision form of the operator-limited rung 3 at the edges of its
tiles: column-tile groups of one to four tiles (two for the div tiles at 8
targets), sample counts around the 32-sample chunks, every padded target
count, and rung-2 operators of every row kind (products and quotients, sums,
differences, unary).  Selections against the FP64 oracle (the selected
scores are rescored in FP64: check_selection's bound)."""
import numpy as np
import pytest

from tests.checks import check_selection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,T,ops2", [
    (4, 31, 1, ("mul", "add")), (9, 32, 2, ("div", "sub")), (17, 33, 8, ("mul", "rdiv")),
    (26, 64, 7, ("sq", "mul", "div")), (26, 65, 1, ("inv", "sub", "mul")), (33, 96, 4, ("mul", "sqrt")),
    (18, 20, 12, ("exp", "log", "mul")), (8, 5, 1, ("mul",)), (26, 40, 3, ("add", "rdiv"))])
@pytest.mark.parametrize("mode", ["per_target", "max"])
def test_tile_edges(oracle_mod, p, n, T, ops2, mode):
    import torch
    import paper_2602_06986_amd as D
    O = oracle_mod
    rng = np.random.default_rng(1000 * p + n)
    X = rng.lognormal(0, 0.4, size=(p, n))
    Y = np.array([X[0] * X[1] * X[2] / X[3] + 0.2 * X[t % p] + 0.1 * rng.normal(size=n) for t in range(T)])
    rung_ops = [None, ("sq",), ops2, ("mul", "div", "rdiv")]
    rung_pool = [None, None, None, 0]
    q = D.params(rung=3, k=12, rung_ops=rung_ops, rung_pool=rung_pool, precision=D.BF16_GUARD,
                 score_mode=D.SCORE_MAX if mode == "max" else D.SCORE_PER_TARGET)
    sp = O.Space(p, 3, O.OPS, rung_ops, rung_pool)
    lists, _, nvalid = O.sis(sp, X, None, Y, 12, (), mode)
    c = D.Context(0)
    try:
        ids, sc, _, st = c.generate_screen(torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda"), q)
        assert st["n_scored"] == nvalid
        for t in range(len(lists)):
            check_selection(ids[t].cpu().numpy(), sc[t].cpu().numpy(), lists[t][0], lists[t][1], what="list %d" % t)
    finally:
        c.close()


@pytest.mark.parametrize("narrow", [0, 3, 7, 10])
@pytest.mark.parametrize("k,dedup", [(1, True), (40, True), (40, False)])
def test_bounds_in_the_pool(oracle_mod, narrow, k, dedup):
    """Pools in which no, some, most or all of the best candidates hold upper
    bounds of their scores (columns narrow about their mean are too
    ill-conditioned for BF16 scores): rescoring in stages gives the selection
    of the exact scores."""
    import torch
    import paper_2602_06986_amd as D
    O = oracle_mod
    p, n = 10, 150
    rng = np.random.default_rng(77 + narrow)
    X = rng.lognormal(0, 0.6, size=(p, n))
    X[:narrow] = 1.0 + 0.15 * (X[:narrow] - X[:narrow].mean(1, keepdims=True))
    Y = np.array([X[0] * X[5] + X[9] / X[2] + 0.02 * rng.normal(size=n)])
    rung_ops = [None, ("sq",), ("mul", "add"), ("mul", "div")]
    rung_pool = [None, None, None, 0]
    sp = O.Space(p, 3, O.OPS, rung_ops, rung_pool)
    lists, _, nvalid = O.sis(sp, X, None, Y, k, (), "per_target", dedup=dedup)
    every = O.screen_scores(sp, X, Y, None, "per_target")[0]
    q = D.params(rung=3, k=k, rung_ops=rung_ops, rung_pool=rung_pool, precision=D.BF16_GUARD, dedup=dedup)
    c = D.Context(0)
    try:
        for _ in range(2):                   # the second call starts from settled sizes
            ids, sc, _, st = c.generate_screen(torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda"), q)
        assert st["n_scored"] == nvalid
        check_selection(ids[0].cpu().numpy(), sc[0].cpu().numpy(), lists[0][0], lists[0][1],
                        None if dedup else every[0])
    finally:
        c.close()
