"""OMP and the model ranking at the sizes where their kernels change course:
rows kept in registers or re-read (2048 samples), odd row counts (two rows
per wave), every model size, warm starts with rows dropped, more problems
than one launch takes (16), short and long bands.  Tolerances are the parity
bar: 1e-10 of the largest coefficient and of the RMSE."""
import ctypes as C
import math

import numpy as np
import pytest

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


def dev(torch, a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def _problem(seed, S, n, D):
    rng = np.random.default_rng(seed)
    F = rng.normal(size=(S, n)) + 0.7 * rng.normal(size=n) + rng.uniform(-3, 3, size=(S, 1))
    y = 1.0 + sum((1.5 - 0.1 * j) * F[(7 * j) % S] for j in range(D)) + rng.normal(size=n)
    return F, rng.permutation(10 * S)[:S].astype(np.int64), y


def _check(got, want, y):
    act, coef, rmse, res = got
    act_o, coef_o, rmse_o, res_o = want
    k = len(act_o)
    assert list(act[:k]) == list(act_o) and all(v == -1 for v in act[k:])
    assert np.max(np.abs(coef[:k + 1] - coef_o)) <= 1e-10 * np.max(np.abs(coef_o))
    assert abs(rmse - rmse_o) <= 1e-10 * rmse_o + 1e-13 * np.std(y)
    assert np.max(np.abs(res - res_o)) <= 1e-10 * np.max(np.abs(y))


@pytest.mark.parametrize("S,n,D", [(1, 3, 1), (8, 10, 8), (9, 511, 3), (33, 512, 8), (40, 513, 5), (257, 2047, 6),
                                   (64, 2048, 8), (65, 2049, 7), (31, 5000, 4), (2051, 100, 2)])
def test_omp_sizes(torch, ctx, oracle_mod, S, n, D):
    F, ids, y = _problem(S + n, S, n, min(D, 3))
    out = ctx.omp(dev(torch, F), dev(torch, ids), dev(torch, y), D)
    _check([t.cpu().numpy() if i != 2 else float(t[0]) for i, t in enumerate(out)], oracle_mod.omp(F, ids, y, D), y)


@pytest.mark.parametrize("init,kept", [((4, 4, 90), (4,)), ((0, 1, 2, 3, 4, 5, 6, 7), (0, 1, 2, 3, 4, 5, 6, 7)),
                                       ((-1, 30, 2), (30, 2))])
def test_omp_warm_start(torch, ctx, oracle_mod, init, kept):
    F, ids, y = _problem(5, 60, 300, 3)
    F[11] = 2.5                                     # a constant row is never picked
    D = 8
    it = torch.as_tensor(np.array(init, np.int32), device="cuda")
    out = ctx.omp(dev(torch, F), dev(torch, ids), dev(torch, y), D, it)
    want = oracle_mod.omp(F, ids, y, D - (len(init) - len(kept)), kept)
    _check([t.cpu().numpy() if i != 2 else float(t[0]) for i, t in enumerate(out)], want, y)


@pytest.mark.parametrize("fn", ["discover_omp", "discover_omp_noalloc"])
def test_omp_many_problems(torch, ctx, oracle_mod, fn):
    import paper_2602_06986_amd as Dm
    nb, D = 19, 3
    data = [_problem(100 + b, 3 + 5 * b, 20 + 13 * b, 2) for b in range(nb)]
    devs = [tuple(dev(torch, v) for v in d) for d in data]
    ldr = max(d[0].shape[1] for d in data)
    act = torch.empty((nb, D), dtype=torch.int32, device="cuda")
    coef = torch.empty((nb, D + 1), dtype=torch.float64, device="cuda")
    rmse = torch.empty(nb, dtype=torch.float64, device="cuda")
    res = torch.empty((nb, ldr), dtype=torch.float64, device="cuda")
    pbs = (Dm.L0Problem * nb)()
    for b, (F, ids, y) in enumerate(devs):
        pbs[b].n, pbs[b].S, pbs[b].F, pbs[b].ldf = F.shape[1], F.shape[0], F.data_ptr(), F.shape[1]
        pbs[b].ids, pbs[b].y = ids.data_ptr(), y.data_ptr()
    for with_resid in (True, False):
        Dm._check(getattr(Dm.lib(), fn)(ctx.h, pbs, nb, D, None, 0, act.data_ptr(), coef.data_ptr(), rmse.data_ptr(),
                                        res.data_ptr() if with_resid else None, ldr,
                                        C.c_void_p(torch.cuda.current_stream().cuda_stream)))
        torch.cuda.synchronize()
        for b, (F, ids, y) in enumerate(data):
            _check([act[b].cpu().numpy(), coef[b].cpu().numpy(), float(rmse[b]), res[b, :len(y)].cpu().numpy()],
                   oracle_mod.omp(F, ids, y, D), y)


@pytest.mark.parametrize("copies,m", [(1, 3), (20, 64), (31, 40), (70, 64)])
def test_ranking_of_short_and_long_bands(torch, ctx, oracle_mod, copies, m):
    """Bands of one to some thousand tied subsets: rows repeated `copies`
    times give copies^2 equal models, ordered by their ID tuples."""
    rng = np.random.default_rng(copies)
    n = 120
    A, B = rng.normal(size=n), rng.normal(size=n)
    F = np.vstack([np.tile(A, (copies, 1)), np.tile(B, (copies, 1)), rng.normal(size=(6, n))])
    ids = rng.permutation(9000)[:len(F)].astype(np.int64)
    y = A - 2.0 * B + 0.3 * rng.normal(size=n)
    want = oracle_mod.l0(F, ids, y, 2, m)
    sub, rmse, coef, res, st = ctx.l0_fit(dev(torch, F), dev(torch, ids), dev(torch, y), 2, m)
    sub, rmse, res = sub.cpu().numpy(), rmse.cpu().numpy(), res.cpu().numpy()
    assert st["n_band"] >= min(m, copies * copies)
    for q, w in enumerate(want):
        assert sorted(ids[sub[q]]) == sorted(int(v) for v in w["ids"]), q
        assert abs(rmse[q] - w["rmse"]) <= 1e-10 * w["rmse"]
        assert np.max(np.abs(res[q] - w["resid"])) <= 1e-10 * np.max(np.abs(y))
