"""The FP64 pair screen in its matrix form: tile shapes, ragged sample
counts, target counts, operator subsets, and data at the limits of
unshifted moments (narrow columns, huge and tiny scales, zeros, near
cancellation), where candidates go to the exact fix-up or the whole
problem to the vector form.  Selections against the FP64 oracle; scores to
1e-10 relative."""
import numpy as np
import pytest

from tests.checks import check_selection

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.fixture(scope="module")
def ctx(torch):
    import paper_2602_06986_amd as D
    c = D.Context(0)
    yield c
    c.close()


def _data(kind, p, n, T, seed):
    rng = np.random.default_rng(seed)
    X = rng.uniform(0.5, 2.0, size=(p, n))
    if kind == "narrow":                     # every column within 0.1 % of its mean: vector form
        X = 300.0 + 0.1 * rng.normal(size=(p, n))
    elif kind == "one_narrow":               # products of two narrow features by the fix-up
        X[1] = 300.0 + 0.1 * rng.normal(size=n)
    Z = (X - X.mean(1, keepdims=True)) / X.std(1, keepdims=True)
    Y = np.stack([Z[t % p] * Z[(t + 1) % p] + 0.5 * Z[(3 * t + 2) % p] + 0.2 * rng.normal(size=n) for t in range(T)])
    if kind == "huge":
        X[2] *= 1e60
        X[3] *= 1e-60
    elif kind == "tiny":                     # squares of products underflow
        X *= 1e-100
    elif kind == "zeros":
        X[0, ::3] = 0.0
        X[1] -= 1.0
    elif kind == "near":                     # sums and differences that almost cancel
        X[1] = X[0] * (1.0 + 1e-9 * rng.normal(size=n))
        X[2] = -X[0] + 1e-3 * rng.normal(size=n)
    elif kind == "overflow":
        X[3] = 700.0 + rng.uniform(0, 9, size=n)
    return X, Y


def _check(torch, ctx, O, X, Y, mode="per_target", k=20, units=None, dedup=True, **prm):
    import paper_2602_06986_amd as D
    T = len(Y)
    w = {"X": X, "Y": Y, "units": units, "p": X.shape[0], "n": X.shape[1], "T": T,
         "B": 0 if units is None else units.shape[1], "ops": prm.get("ops", D.OPS), "rung": 2, "rung_ops": None,
         "rung_pool": None}
    sp = O.Space.of(w)
    lists, status, nvalid = O.sis(sp, X, units, Y, k, (), mode, dedup=dedup)
    every = O.screen_scores(sp, X, Y, units, mode)[0]      # (duplicates tie at the cut where they are kept)
    q = D.params(rung=2, k=k, score_mode=D.SCORE_MAX if mode == "max" else D.SCORE_PER_TARGET, dedup=dedup, **prm)
    for _ in range(2):                       # the second call starts from settled sizes
        ids, sc, _, st = ctx.generate_screen(torch.as_tensor(X, device="cuda"), torch.as_tensor(Y, device="cuda"), q,
                                             units=units)
    assert st["n_scored"] == nvalid
    for t in range(len(lists)):
        check_selection(ids[t].cpu().numpy(), sc[t].cpu().numpy(), lists[t][0], lists[t][1],
                        None if dedup else every[t], what="list %d" % t)


@pytest.mark.parametrize("p,n,T,mode", [
    (4, 15, 1, "per_target"), (5, 16, 2, "per_target"), (6, 17, 16, "per_target"), (7, 64, 5, "max"),
    (9, 65, 3, "max"), (10, 129, 1, "per_target"), (11, 33, 1, "per_target"), (12, 40, 4, "max"),
    (13, 31, 8, "max"), (16, 20, 8, "max"), (19, 25, 1, "per_target"), (14, 24, 2, "max")])
def test_sizes(torch, ctx, oracle_mod, p, n, T, mode):
    X, Y = _data("plain", p, n, T, 100 * p + n)
    _check(torch, ctx, oracle_mod, X, Y, mode)


@pytest.mark.parametrize("kind", ["narrow", "one_narrow", "huge", "tiny", "zeros", "near", "overflow"])
@pytest.mark.parametrize("T", [1, 3])
def test_data_limits(torch, ctx, oracle_mod, kind, T):
    X, Y = _data(kind, 8, 77, T, 7)
    # (the oracle's duplicate test squares a product of two sums of squares)
    _check(torch, ctx, oracle_mod, X, Y, dedup=kind not in ("huge", "tiny"))


@pytest.mark.parametrize("ops", [("mul",), ("add", "sub"), ("div",), ("rdiv", "sub"), ("sq", "add", "rdiv")])
def test_operator_subsets(torch, ctx, oracle_mod, ops):
    X, Y = _data("plain", 9, 50, 2, 3)
    _check(torch, ctx, oracle_mod, X, Y, ops=ops, k=10)


def test_units(torch, ctx, oracle_mod):
    X, Y = _data("plain", 9, 90, 2, 5)
    U = np.array([[0, 0]] * 3 + [[1, 0]] * 2 + [[0, 1]] * 2 + [[1, -1]] * 2, dtype=np.int32)
    _check(torch, ctx, oracle_mod, X, Y, units=U)


def test_batch_of_both_forms(torch, ctx, oracle_mod):
    """One call over datasets of which some take the matrix form and some
    the vector form equals the calls apart."""
    import paper_2602_06986_amd as D
    q = D.params(rung=2, k=15)
    data = [_data(kind, p, n, 1, 40 + p) for kind, p, n in (("plain", 8, 60), ("narrow", 7, 45), ("plain", 11, 130),
                                                            ("narrow", 6, 33), ("zeros", 9, 70))]
    Xs = [torch.as_tensor(X, device="cuda") for X, _ in data]
    Ys = [torch.as_tensor(Y, device="cuda") for _, Y in data]
    both = ctx.generate_screen_batch(Xs, Ys, q)
    for b in range(len(data)):
        ids, sc, vals, st = ctx.generate_screen(Xs[b], Ys[b], q)
        assert torch.equal(ids, both[b][0]) and torch.equal(sc, both[b][1]) and torch.equal(vals, both[b][2])
        assert st["n_scored"] == both[b][3]["n_scored"]
