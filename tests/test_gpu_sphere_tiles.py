"""Spherical stage tiles past one per CU: every phase loads what it needs."""
import numpy as np
import pytest

from parity import rel_errors, state_rel
from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [("f64", 124), ("f64", 125), ("f32", 176), ("f32", 181)])
def test_many_tiles_match_oracle(orc, prec, n):
    """The last size with all loads at once and the first without, ragged in
    both directions: FP64 to 1e-12 per variable and FP32 to 1e-5 of the state,
    as on small grids."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from oracle import sphere as S
    from paper_2602_08670_amd import fv

    steps = 4
    kw = dict(flux=0, recon=0, rk_stages=2, g=1.0, omega=0.5)
    cen, *_ = S.geometry(S.Config(n=n))
    q0 = I.sphere_state(cen, seed=5, u0=0.3, omega=0.5)
    print(f"[sphere tiles] {prec} n={n}", flush=True)
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
