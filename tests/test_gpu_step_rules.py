"""Each kernel that a step in one launch can be, against a launch per stage."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(58, 11), (61, 509), (113, 680)])
@pytest.mark.parametrize("prec,flux,recon,rk", [
    ("f32", "rusanov", "minmod", 2), ("f32", "roe", "minmod", 2), ("f32", "hlle", "first", 2), ("f32", "hlle", "minmod", 3),
    ("f32", "rusanov", "first", 3), ("f64", "roe", "minmod", 2), ("f64", "hlle", "first", 2), ("f64", "hlle", "minmod", 3),
])
@pytest.mark.parametrize("eqn,fixed", [("swe_bed", False), ("swe", True), ("euler", False), ("euler", True)])
def test_same_bits_as_a_launch_per_stage(eqn, fixed, prec, flux, recon, rk, nx, ny):
    """Four steps in one call against four calls of one step, walls in x:
    equal bits.  Tiles of 60 columns for two stages and 56 for three: the
    first size takes 4 rows of cells each; the second 8 (FP64 with three stages
    256 tiles of 4, the most that go in one launch); the third 8, just within
    256 tiles for two stages (three take a launch per stage)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    rng = np.random.default_rng(nx + ny)
    shape = (ny, nx)
    b = None
    if eqn == "euler":
        r, u, v, p = 1 + 0.2 * rng.random(shape), *(0.1 * rng.standard_normal((2, *shape))), 1 + 0.2 * rng.random(shape)
        q = np.stack([r, r * u, r * v, p / 0.4 + 0.5 * r * (u * u + v * v)])
    else:
        q = np.stack([1 + 0.2 * rng.random(shape), *(0.1 * rng.standard_normal((2, *shape)))])
        b = 0.1 * rng.random(shape) if eqn == "swe_bed" else None
    dt = np.float64 if prec == "f64" else np.float32
    print(f"[step rules] {prec} {flux} {recon} rk{rk} {eqn} fixed={fixed} {nx}x{ny}", flush=True)
    runs = []
    for calls in ([4], [1] * 4):
        s = fv.Solver(q.astype(dt), None if b is None else b.astype(dt), prec=fv.FV_F64 if prec == "f64" else fv.FV_F32,
                      bc_x=fv.FV_BC_WALL, lx=1.0, ly=ny / nx, rk_stages=rk, cfl=0.3, dt_fixed=0.05 / nx if fixed else 0.0,
                      flux={"hlle": fv.FV_FLUX_HLLE, "rusanov": fv.FV_FLUX_RUSANOV, "roe": fv.FV_FLUX_ROE}[flux],
                      recon=fv.FV_RECON_MINMOD if recon == "minmod" else fv.FV_RECON_FIRST)
        for k in calls:
            s.run(k)
        runs.append((s.state(), s.time()))
        s.close()
    assert np.isfinite(runs[0][0]).all() and np.abs(runs[0][0] - q).max() > 0
    assert np.array_equal(runs[0][0], runs[1][0])
    assert runs[0][1] == runs[1][1]
