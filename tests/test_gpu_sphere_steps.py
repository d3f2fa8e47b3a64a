"""Spherical steps whose end is more than one launch's business: one-stage
steps over many tiles, and a step that fails."""
import ctypes

import numpy as np
import pytest

from parity import rel_errors, state_rel
from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu

N = 400  # 800 x 400 cells: 1250 tiles


@pytest.fixture(scope="module")
def fv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv as F

    return F


def state(S):
    cen, *_ = S.geometry(S.Config(n=N))
    return I.sphere_state(cen, seed=5, u0=0.3, omega=0.5)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_one_stage_steps(orc, fv, prec):
    """A tile reads its neighbours' cells of the step's start, however late it
    runs: fixed Delta t, FP64 to 1e-12 per variable, FP32 to 1e-5 of the state,
    against the oracle."""
    from oracle import sphere as S

    q0 = state(S)
    kw = dict(flux=0, recon=0, rk_stages=1, g=1.0, omega=0.5, dt_fixed=2.0 ** -11)
    print(f"[sphere steps] {prec} one stage", flush=True)
    s = fv.SphereSolver(q0, prec=fv.FV_F64 if prec == "f64" else fv.FV_F32, **kw)
    s.run(4)
    t, k = s.time()
    out = s.state()
    s.close()
    ref, t_ref, rc = S.run(S.Config(n=N, nthreads=8, **kw), q0, 4)
    assert rc == 0 and k == 4 and t == t_ref
    if prec == "f64":
        assert np.all(rel_errors(out, ref) <= 1e-12)
    else:
        assert state_rel(out, ref) <= 1e-5


@pytest.mark.parametrize("rk", [1, 2])
def test_failing_step(orc, fv, rk):
    """Delta t four times the stable one, from two steps before the depth turns
    negative: the third step fails and is counted, no tile of it keeps the cells
    of the step before, and nothing follows, however the steps are called.
    (Near a vanishing depth the failing step amplifies rounding without bound,
    so its values are not compared with the oracle's.)"""
    from oracle import sphere as S

    cfg = S.Config(n=N, nthreads=8, g=1.0, omega=0.5, rk_stages=rk)
    states = [state(S)]
    dt = 4 * S.lib().sph_dt(cfg._c(), S._dp(np.ascontiguousarray(states[0])))
    cfg = S.Config(n=N, nthreads=8, g=1.0, omega=0.5, rk_stages=rk, dt_fixed=dt)
    rc = 0
    while rc == 0 and len(states) < 60:
        q, _, rc = S.run(cfg, states[-1], 1)
        states.append(q)
    assert rc != 0 and len(states) > 4
    print(f"[sphere steps] rk{rk} fails at step {len(states) - 1}", flush=True)

    def run(calls):
        s = fv.SphereSolver(states[-4], prec=fv.FV_F64, flux=0, recon=0, rk_stages=rk, g=1.0, omega=0.5, dt_fixed=dt)
        for k in calls:
            s.run(k)
        t, n = ctypes.c_double(), ctypes.c_int64()
        rc = fv.lib.fv_sphere_time(s.h, ctypes.byref(t), ctypes.byref(n))
        out = s.state()
        s.close()
        return out, n.value, rc

    before, n, rc = run([2])
    assert rc == fv.FV_OK and n == 2
    out, n, rc = run([3])
    assert rc == fv.FV_E_INADMISSIBLE and n == 3
    kept = (out == before).all(axis=0).reshape(N // 4, 4, 2 * N // 32, 32).all(axis=(1, 3))
    assert not kept.any()
    for calls in ([6], [1, 1, 1, 1], [2, 3]):
        o, n, rc = run(calls)
        assert rc == fv.FV_E_INADMISSIBLE and n == 3 and np.array_equal(o, out, equal_nan=True)
