"""The pair form of the branch-and-bound leaves below parents of two and
three rows (four and five terms), over its steps of 64 leaves and its 32
children per wave: against every subset's residual from the correlations,
formed in numpy by elimination."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _all_rss(F, y, D):
    """Every subset of D rows (in lexicographic order) and its RSS (NaN where singular)."""
    S, n = F.shape
    Z = F - F.mean(1, keepdims=True)
    s = np.sqrt((Z * Z).sum(1))
    Z = Z / np.where(s > 0, s, 1.0)[:, None]
    yc = y - y.mean()
    G, c = Z @ Z.T, Z @ yc
    sub = np.array(list(itertools.combinations(range(S), D)), dtype=np.int32)
    M = G[sub[:, :, None], sub[:, None, :]]
    b = c[sub]
    rss = np.full(len(sub), yc @ yc)
    ok = np.ones(len(sub), bool)
    for k in range(D):
        piv = M[:, k, k].copy()
        ok &= piv > 1e-10
        piv[~ok] = 1.0
        rss -= b[:, k] ** 2 / piv
        f = M[:, k + 1:, k] / piv[:, None]
        b[:, k + 1:] -= f * b[:, k, None]
        M[:, k + 1:, k + 1:] -= f[:, :, None] * M[:, None, k, k + 1:]
    rss[~ok] = np.nan
    return sub, rss


@pytest.mark.parametrize("S,D", [(33, 4), (65, 4), (68, 4), (32, 5), (35, 5)])
@pytest.mark.parametrize("m", [1, 6])
@pytest.mark.parametrize("planted", [False, True])
def test_deep_leaves(S, D, m, planted):
    import torch
    import paper_2602_06986_amd as Dm
    rng = np.random.default_rng(100 * S + 10 * D + m)
    n = 150
    F = rng.normal(size=(S, n))
    F[S // 2] = F[3]                             # a duplicate: singular subsets
    F[S // 3] = 1.0                              # a constant row
    y = rng.normal(size=n) * (0.3 if planted else 1.0)
    if planted:
        y = y + F[0] - 0.8 * F[S - 1] + 0.5 * F[S // 4] + 0.4 * F[5]
    sub, rss = _all_rss(F, y, D)
    best = np.argsort(rss)[:m + 1]
    # (the m best are apart by more than rounding, except through the duplicate row)
    rmse = np.sqrt(rss / n)
    ids = rng.permutation(10 ** 6)[:S].astype(np.int64)
    c = Dm.Context(0)
    try:
        s, r, _, _, _ = c.l0_bnb(*[torch.as_tensor(a, device="cuda") for a in (F, ids, y)], D, m)
        s, r = s.cpu().numpy(), r.cpu().numpy()
    finally:
        c.close()
    place = {tuple(t): e for e, t in enumerate(sub.tolist())}
    seen = [place[tuple(sorted(t.tolist()))] for t in s]
    assert len(set(seen)) == m
    for q in range(m):
        assert abs(r[q] - rmse[seen[q]]) <= 1e-10 * r[q]
        assert abs(r[q] - rmse[best[q]]) <= 1e-10 * r[q]
