"""The Gram product of the L0 methods at the edges of its chunks of 32
samples, its four runs per block and its 32 x 32 tiles: models of the pair
sweep against a direct FP64 least squares over all pairs (RMSE to 1e-10 of
the best fit, subsets equal)."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,n", [(3, 5), (15, 16), (16, 17), (31, 31), (32, 33), (33, 48), (40, 63), (24, 64),
                                 (63, 65), (47, 127), (20, 129), (34, 257)])
def test_edges(S, n):
    import torch
    import paper_2602_06986_amd as D
    rng = np.random.default_rng(1000 * S + n)
    F = rng.normal(size=(S, n)) + rng.normal(size=(S, 1))
    y = F[0] - 0.7 * F[S - 1] + 0.3 * rng.normal(size=n)
    best = None
    for a, b in itertools.combinations(range(S), 2):
        A = np.stack([np.ones(n), F[a], F[b]], axis=1)
        r = y - A @ np.linalg.lstsq(A, y, rcond=None)[0]
        v = float(np.sqrt(r @ r / n))
        if best is None or v < best[0]:
            best = (v, a, b)
    c = D.Context(0)
    try:
        ids = np.arange(S, dtype=np.int64)
        sub, rmse, _, _, _ = c.l0_fit(*(torch.as_tensor(x, device="cuda") for x in (F, ids, y)), 2, 1)
        assert sorted(sub[0].cpu().numpy().tolist()) == [best[1], best[2]]
        assert abs(float(rmse[0]) - best[0]) <= 1e-10 * best[0] + 1e-12 * np.std(y)
    finally:
        c.close()
