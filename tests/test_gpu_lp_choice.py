"""Which kernel takes the pair candidates of a precision form: the one that
is faster for the shape, from the first call on, under every tile width and
schedule (one operand feature per wave takes a third of the BF16 kernel's
time at these shapes, the matrix form less)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,T", [(8, 300, 3), (12, 1000, 8)])
def test_faster_form(p, n, T):
    import torch
    import paper_2602_06986_amd as D
    rng = np.random.default_rng(4)
    X = rng.lognormal(0.0, 0.3, size=(p, n))
    Y = np.array([X[3] * X[4] * X[5] + 0.1 * rng.normal(size=n) for t in range(T)])
    Xd, Yd = torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda")
    c = D.Context(0)
    try:
        ref = None
        for tile_j, sched in ((0, 0), (1, 0), (0, -1), (1, -1), (0, 0)):
            q = D.params(rung=2, k=12, precision=D.BF16_GUARD, score_mode=D.SCORE_MAX, tile_j=tile_j, sched=sched)
            for _ in range(3):
                ids, sc, _, st = c.generate_screen(Xd, Yd, q)
                assert st["tile_j"] > 0      # the FP64 kernels ran
                ref = ref or (ids, sc)
                assert torch.equal(ids, ref[0]) and torch.equal(sc, ref[1])
    finally:
        c.close()
