"""The pair form of the branch-and-bound leaves at the edges of its steps:
row counts around its steps of 64 leaves, its 32 children per wave and 128
per block, few parents and many, on targets of pure noise (weak cuts: whole
branches are stepped through) and planted ones (branches end within a
step).  Models equal the exhaustive search's (RMSE to 1e-10, as its tests)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2602_06986_amd as D
    c = D.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("S", [3, 33, 64, 65, 66, 129, 130, 193, 260])
@pytest.mark.parametrize("D,m", [(2, 1), (2, 7), (3, 1), (3, 5)])
@pytest.mark.parametrize("planted", [False, True])
def test_steps(ctx, S, D, m, planted):
    import torch
    rng = np.random.default_rng(100 * S + 10 * D + m)
    n = 150
    F = rng.normal(size=(S, n))
    if S > 40:
        F[S // 2] = F[3]                         # a duplicate: singular pairs
        F[S // 3] = 1.0                          # a constant row
    y = rng.normal(size=n) * (0.3 if planted else 1.0)
    if planted:
        y = y + F[0] - 0.8 * F[S - 1] + 0.5 * F[S // 4]
    ids = rng.permutation(10 ** 6)[:S].astype(np.int64)
    m = min(m, math.comb(S, D))
    d = [torch.as_tensor(a, device="cuda") for a in (F, ids, y)]
    s1, r1, _, _, _ = ctx.l0_fit(*d, D, m)
    s2, r2, _, _, _ = ctx.l0_bnb(*d, D, m)
    for q in range(m):
        assert sorted(ids[s1[q].cpu().numpy()].tolist()) == sorted(ids[s2[q].cpu().numpy()].tolist()), q
        assert abs(float(r1[q]) - float(r2[q])) <= 1e-10 * float(r1[q]) + 1e-13 * np.std(y)
