"""Spherical stage kernels on both sides of the rule on tiles per CU."""
import numpy as np
import pytest

from parity import rel_errors, state_rel
from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flux,recon,rk", [("hlle", 0, 2), ("roe", 0, 3), ("rusanov", 1, 2), ("roe", 1, 1)])
@pytest.mark.parametrize("prec,n", [("f64", 128), ("f64", 129), ("f32", 176), ("f32", 177)])
def test_both_sides_match_oracle(orc, prec, n, flux, recon, rk):
    """FP64 tiles of 32 x 4 cells: 256 at n = 128, 297 at 129; FP32 of 32 x 8:
    242 at n = 176, 276 at 177 (ceil(2 n / 32) ceil(n / rows), 256 the last with
    all loads at once).  FP64 to 1e-12 per variable, FP32 to 1e-5 of the state,
    as on small grids."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from oracle import sphere as S
    from paper_2602_08670_amd import fv

    steps = 3
    fl = {"hlle": fv.FV_FLUX_HLLE, "rusanov": fv.FV_FLUX_RUSANOV, "roe": fv.FV_FLUX_ROE}[flux]
    kw = dict(flux=fl, recon=recon, rk_stages=rk, g=1.0, omega=0.5)
    cen, *_ = S.geometry(S.Config(n=n))
    q0 = I.sphere_state(cen, seed=5, u0=0.3, omega=0.5)
    print(f"[sphere rules] {prec} n={n} {flux} recon={recon} rk{rk}", flush=True)
    s = fv.SphereSolver(q0, prec=fv.FV_F64 if prec == "f64" else fv.FV_F32, **kw)
    s.run(steps)
    t, k = s.time()
    out = s.state()
    s.close()
    ref, t_ref, rc = S.run(S.Config(n=n, nthreads=8, **kw), q0, steps)
    assert rc == 0 and k == steps
    if prec == "f64":
        assert abs(t - t_ref) <= 1e-13 * t_ref
        assert np.all(rel_errors(out, ref) <= 1e-12)
    else:
        assert abs(t - t_ref) <= 1e-5 * t_ref
        assert state_rel(out, ref) <= 1e-5
