"""The tile shapes of the stage kernels: a grid's size picks the shape, and a
cell's arithmetic is the same in each."""
import numpy as np
import pytest

from parity import max_rel, state_rel
from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv as F

    return F


def run(fv, q, b, steps, **kw):
    print(f"[shape] {np.shape(q)} bed={b is not None} {kw}", flush=True)
    s = fv.Solver(q, b, **kw)
    s.run(steps)
    t, n = s.time()
    assert n == steps
    out = s.state()
    s.close()
    return out, t


@pytest.mark.parametrize("eq", ["swe", "swe_bed", "euler"])
@pytest.mark.parametrize("copies", [7, 13, 28])
def test_periodic_copies_bitwise(fv, eq, copies):
    """A periodic 64^2 solve (4-row tiles) and the same data repeated over a
    grid of the next shapes (448^2, 832^2, 1792^2 cells): the same bits in
    every copy."""
    if eq == "euler":
        q, b = I.random_smooth_euler(64, seed=3), None
    else:
        q, b = I.swe_bathy(64, seed=2)
        b = b if eq == "swe_bed" else None
        q[1] = 0.05 * np.sin(2 * np.pi * np.arange(64) / 64)[None, :]
    small, t0 = run(fv, q, b, 3, h_ref=1.0)
    rep = (1, copies, copies)
    big, t1 = run(fv, np.tile(q, rep), None if b is None else np.tile(b, rep[1:]), 3, h_ref=1.0, lx=float(copies),
                  ly=float(copies))
    assert t0 == t1
    assert np.array_equal(big, np.tile(small, rep))


@pytest.mark.parametrize("nx,ny", [(5, 4), (63, 5), (65, 401), (399, 401), (401, 405), (819, 1003)])
@pytest.mark.parametrize("eq,bc", [("swe_bed", (1, 1)), ("swe", (0, 1)), ("euler", (1, 0))])
def test_ragged_grids(fv, orc, nx, ny, eq, bc):
    """Cut last tiles, grids narrower than a tile and both ghost kinds, two
    steps against the oracle: FP32 state within 1e-5 (rounding of four
    stages is below 1e-6), FP64 per variable within 1e-12."""
    n = max(nx, ny)
    if eq == "euler":
        q, b = I.random_smooth_euler(n, seed=4), None
    else:
        q, b = I.swe_bathy(n, seed=2)
        q[1] = 0.05 * np.sin(np.arange(n) / 5.0)[None, :]
        q[2] = 0.03 * np.cos(np.arange(n) / 3.0)[:, None]
    q = q[:, :ny, :nx].copy()
    b = b[:ny, :nx].copy() if eq == "swe_bed" else None
    for prec, dt in ((fv.FV_F32, np.float32), (fv.FV_F64, np.float64)):
        q0, b0 = q.astype(dt).astype(np.float64), None if b is None else b.astype(dt).astype(np.float64)
        out, t = run(fv, q0, b0, 2, prec=prec, bc_x=bc[0], bc_y=bc[1], lx=1.0, ly=ny / nx)
        cfg = orc.Config(eqn=1 if eq == "euler" else 0, nx=nx, ny=ny, bc_x=bc[0], bc_y=bc[1], lx=1.0, ly=ny / nx,
                         nthreads=8)
        ref, t_ref, *_ = orc.run(cfg, q0, b0, 2)
        if prec == fv.FV_F64:
            assert abs(t - t_ref) <= 1e-13 * t_ref and max_rel(out, ref) <= 1e-12
        else:
            assert abs(t - t_ref) <= 1e-6 * t_ref and state_rel(out, ref) <= 1e-5


@pytest.mark.parametrize("nvar,cx,cy,f", [(1, 1, 1, 1), (3, 300, 2, 1), (3, 37, 5, 7), (4, 9, 3, 32), (2, 3, 2, 256),
                                          (2, 2, 3, 300)])
def test_coarsen_factors(fv, nvar, cx, cy, f):
    """Block averages for factors that fill, cut or exceed a workgroup's
    columns: the mean rounded to float once."""
    import torch

    x = torch.rand((nvar, cy * f, cx * f), device="cuda", generator=torch.Generator("cuda").manual_seed(f)) + 0.5
    ref = x.double().cpu().numpy().reshape(nvar, cy, f, cx, f).mean(axis=(2, 4))
    got = fv.coarsen(x, f).double().cpu().numpy()
    assert got.shape == ref.shape and np.abs(got - ref).max() <= 1.2e-7 * ref.max()
