"""Rung 3 over primaries with zeros: quotients by a feature with a zero are
never finite and are left out by the precision form as by the FP64 form (no
longer list of candidates for the exact fix-up), for rung-2 features of
every row kind (products and quotients, sums and differences, unary)."""
import numpy as np
import pytest

from tests.checks import check_selection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zeros", [1, 2])
@pytest.mark.parametrize("ops2,n,T", [(("mul", "div"), 60, 2), (("add", "sub"), 33, 1), (("rdiv", "sq", "log"), 65, 8),
                                      (("mul", "sub", "exp", "log"), 60, 2), (("sub", "sqrt", "inv"), 31, 4)])
def test_zero_divisors(oracle_mod, zeros, ops2, n, T):
    import torch
    import paper_2602_06986_amd as D
    O = oracle_mod
    p, k = 10, 12
    rng = np.random.default_rng(4)
    X = rng.lognormal(0.0, 0.3, size=(p, n))
    X[:zeros, ::7] = 0.0
    if "sub" in ops2:
        X[2, 5] = X[3, 5]                    # a difference of positive columns with one zero
    Y = np.array([X[3] * X[4] * X[5] / X[6] + 0.1 * rng.normal(size=n) for t in range(T)])
    rung_ops, rung_pool = [None, ("sq",), ops2, ("mul", "div", "rdiv")], [None, None, None, 0]
    lists, _, nvalid = O.sis(O.Space(p, 3, O.OPS, rung_ops, rung_pool), X, None, Y, k, (), "max")
    Xd, Yd = torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda")
    c = D.Context(0)
    try:
        def status(q, cap):
            c.set_fixup_capacity(cap)
            got = c.generate_screen(Xd, Yd, q, device_stats=True)
            torch.cuda.synchronize()
            return D.decode_stats(got[3], D.ScreenStats)[0]["status"]

        q = {pr: D.params(rung=3, k=k, rung_ops=rung_ops, rung_pool=rung_pool, precision=pr, score_mode=D.SCORE_MAX)
             for pr in (D.FP64, D.BF16_GUARD)}
        for pr in q:
            ids, sc, _, st = c.generate_screen(Xd, Yd, q[pr])
            assert st["n_scored"] == nvalid
            check_selection(ids[0].cpu().numpy(), sc[0].cpu().numpy(), lists[0][0], lists[0][1])
        lo, hi = 0, nvalid                   # entries that the FP64 form lists
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if status(q[D.FP64], mid) == 0 else (mid, hi)
        assert status(q[D.BF16_GUARD], hi) == 0
    finally:
        c.close()
