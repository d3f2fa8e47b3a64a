"""A step in one launch: all stages of a tile in one workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


HEUN = ("f32", "hlle", "minmod", 2)


@pytest.mark.parametrize("nx,ny", [(6, 6), (7, 9), (57, 6), (60, 7), (61, 9), (62, 12), (64, 64), (121, 17), (130, 33),
                                   (61, 517), (121, 697)])
@pytest.mark.parametrize("wall", [(0, 0), (1, 1), (1, 0), (0, 1)])
@pytest.mark.parametrize("eqn,bed", [("swe", True), ("swe", False), ("euler", False)])
@pytest.mark.parametrize("scheme", [HEUN, ("f32", "rusanov", "first", 1), ("f32", "roe", "minmod", 3),
                                    ("f64", "hlle", "minmod", 1), ("f64", "rusanov", "minmod", 2),
                                    ("f64", "roe", "first", 3)])
def test_same_bits_as_a_launch_per_stage(scheme, eqn, bed, wall, nx, ny):
    """Six steps in one call (three pairs of single launches) against six
    calls of one step (a launch per stage), and five against five (an odd step
    at the end): the same cells, the same arithmetic, equal bits.  The last two
    sizes take tiles of 8 and, where there are any, 12 rows, the others of 4."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    rng = np.random.default_rng(nx * 100 + ny)
    shape = (ny, nx)
    if eqn == "swe":
        q = np.stack([1 + 0.2 * rng.random(shape), 0.1 * rng.standard_normal(shape), 0.1 * rng.standard_normal(shape)])
        b = 0.1 * rng.random(shape) if bed else None
    else:
        r, u, v, p = 1 + 0.2 * rng.random(shape), *(0.1 * rng.standard_normal((2, *shape))), 1 + 0.2 * rng.random(shape)
        q, b = np.stack([r, r * u, r * v, p / 0.4 + 0.5 * r * (u * u + v * v)]), None
    prec, flux, recon, rk = scheme
    dt = np.float64 if prec == "f64" else np.float32
    print(f"[step launch] {scheme} {eqn} bed={bed} wall={wall} {nx}x{ny}", flush=True)
    bc = [fv.FV_BC_WALL if w else fv.FV_BC_PERIODIC for w in wall]
    for steps in (6, 5):
        runs = []
        for calls in ([steps], [1] * steps):
            kw = dict(eqn=fv.FV_EULER) if eqn == "euler" else {}
            s = fv.Solver(q.astype(dt), None if b is None else b.astype(dt),
                          prec=fv.FV_F64 if prec == "f64" else fv.FV_F32, bc_x=bc[0], bc_y=bc[1], lx=1.0, ly=ny / nx,
                          flux={"hlle": fv.FV_FLUX_HLLE, "rusanov": fv.FV_FLUX_RUSANOV, "roe": fv.FV_FLUX_ROE}[flux],
                          recon=fv.FV_RECON_MINMOD if recon == "minmod" else fv.FV_RECON_FIRST, rk_stages=rk,
                          cfl=0.3, **kw)
            for k in calls:
                s.run(k)
            runs.append((s.state(), s.time()))
            s.close()
        assert np.isfinite(runs[0][0]).all()
        assert np.array_equal(runs[0][0], runs[1][0])
        assert runs[0][1] == runs[1][1]
