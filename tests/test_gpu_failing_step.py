"""A solve that turns inadmissible during a run: the state is the one that the
failing step produced, the step count includes it, later steps are skipped,
however the steps were launched."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv as F

    return F


def solve(fv, q, calls, kw):
    """State, time, steps and whether a step failed, after run(k) for each k."""
    s = fv.Solver(q, **kw)
    for k in calls:
        s.run(k)
    t, n = ctypes.c_double(), ctypes.c_int64()
    rc = fv.lib.fv_time(s.h, ctypes.byref(t), ctypes.byref(n))
    out = s.state()
    s.close()
    assert rc in (fv.FV_OK, fv.FV_E_INADMISSIBLE)
    return out, t.value, n.value, rc != fv.FV_OK


def doomed(fv, n, before, kw):
    """A state whose step number `before` + 1 fails: smooth waves under a
    Delta t several times the stable one, advanced one step at a time until it
    does."""
    y, x = np.mgrid[0:n, 0:n] / n
    dt = np.float64 if kw["prec"] == fv.FV_F64 else np.float32
    h = 1 + 0.3 * np.sin(2 * np.pi * x) * np.cos(2 * np.pi * y)
    q = np.stack([h, 0.4 * h * np.cos(2 * np.pi * y), 0.3 * h * np.sin(2 * np.pi * (x + y))]).astype(dt)
    states = [q]
    for _ in range(60):
        out, _, _, failed = solve(fv, states[-1], [1], kw)
        if failed:
            break
        states.append(out.astype(dt))
    assert failed and len(states) > before
    return states[-1 - before]


def config(fv, prec, flux, recon, rk, n):
    return dict(prec=fv.FV_F64 if prec == "f64" else fv.FV_F32, rk_stages=rk, h_ref=1.0,
                flux={"hlle": fv.FV_FLUX_HLLE, "roe": fv.FV_FLUX_ROE}[flux],
                recon=fv.FV_RECON_MINMOD if recon == "minmod" else fv.FV_RECON_FIRST, dt_fixed=2.0 / (7.0 * n))


def same(a, b):
    return np.array_equal(a[0], b[0], equal_nan=True) and a[1:] == b[1:]


@pytest.mark.parametrize("prec,flux,recon,rk", [("f32", "hlle", "minmod", 1), ("f64", "roe", "first", 1),
                                                ("f32", "hlle", "minmod", 2), ("f64", "hlle", "minmod", 2),
                                                ("f32", "roe", "minmod", 3), ("f64", "hlle", "first", 3)])
@pytest.mark.parametrize("before", [2, 3])
def test_steps_in_pairs(fv, prec, flux, recon, rk, before):
    """The third and the fourth step fails (the first and the second of a pair
    of single launches), then none, one (a pair's second or a step by itself)
    or more follow: the same state, time and count as one step per call."""
    n = 40
    kw = config(fv, prec, flux, recon, rk, n)
    q = doomed(fv, n, before, kw)
    print(f"[failing step] {prec} {flux} {recon} rk{rk} step {before + 1}", flush=True)
    ref = solve(fv, q, [1] * (before + 1), kw)
    assert ref[2] == before + 1 and ref[3]
    assert solve(fv, q, [before], kw)[2:] == (before, False)
    for after in range(5):
        assert same(solve(fv, q, [before + 1 + after], kw), ref), after
        assert same(solve(fv, q, [1] * (before + 1 + after), kw), ref), after
        assert same(solve(fv, q, [before + 1, after], kw), ref), after


@pytest.mark.parametrize("prec,flux,recon,rk,copies", [("f32", "hlle", "minmod", 2, 20),   # one launch per step
                                                       ("f32", "hlle", "minmod", 1, 30),
                                                       ("f32", "hlle", "minmod", 2, 40),   # a launch per stage
                                                       ("f64", "hlle", "minmod", 3, 16)])
def test_more_workgroups_than_fit(fv, prec, flux, recon, rk, copies):
    """A periodic solve of a few workgroups and its data repeated over a grid
    whose workgroups run in several rounds, every copy of which fails in the
    same step: the same state in every copy, whichever failed first."""
    n = 40
    kw = config(fv, prec, flux, recon, rk, n)
    q = doomed(fv, n, 2, kw)
    ref = solve(fv, q, [4], kw)
    assert ref[2] == 3 and ref[3]
    print(f"[failing step] {prec} rk{rk} {n * copies}^2", flush=True)
    rep = (1, copies, copies)
    big = solve(fv, np.tile(q, rep), [4], dict(kw, lx=float(copies), ly=float(copies)))
    assert same(big, (np.tile(ref[0], rep), *ref[1:]))
