"""Euler HLLE faces of the stage kernels in single precision: each side's flux
is weighed by itself, so a strong neighbour leaves no rounding in a flux that
it has no part in, and a face and its mirror image have the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GAMMA = 1.4


@pytest.fixture(scope="module")
def fv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv as F

    return F


def conserved(r, u, v, p):
    return np.stack([r, r * u, r * v, p / (GAMMA - 1) + 0.5 * r * (u * u + v * v)])


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("sign", [-1, 1])
def test_strong_downstream_neighbour(fv, axis, sign):
    """Flow at four times the sound speed to one side, every fourth cell a
    thousand times as dense and as strong: a face's flux is its upstream cell's
    alone.  A weak cell whose upstream cell is weak and whose downstream cell
    is strong: each of the two fluxes that change it (0.4 x 1.1 x up to 1.6 of
    its content) has at most eight roundings of 2^-24, one more in the sum:
    within 1e-6 of double precision (the strong side's rounding would leave
    0.4 x 1000 x 2^-24, 2e-5)."""
    rng = np.random.default_rng(1)
    n, m = 256, 8
    k = np.arange(n) % 4
    s = np.where(k == 0, 1000.0, 1.0)
    r, p = s * rng.uniform(0.8, 1.25, n), s * rng.uniform(0.8, 1.25, n)
    un = sign * 4 * np.sqrt(GAMMA * p / r).max() * rng.uniform(0.95, 1.05, n)
    ut = rng.uniform(-0.5, 0.5, n)
    u, v = (un, ut) if axis == 0 else (ut, un)
    shape = (m, n) if axis == 0 else (n, m)
    q = conserved(r, u, v, p).astype(np.float32)
    q = np.ascontiguousarray(np.broadcast_to(q[:, None, :] if axis == 0 else q[:, :, None], (4, *shape)))
    lam = 0.4 / (np.abs(un) + np.sqrt(GAMMA * p / r)).max()
    dt = float(np.float32(lam / n))
    print(f"[euler faces] axis {axis} sign {sign}", flush=True)
    sol = fv.Solver(q, prec=fv.FV_F32, recon=fv.FV_RECON_FIRST, rk_stages=1, dt_fixed=dt, lx=shape[1] / n,
                    ly=shape[0] / n, gamma=GAMMA)
    sol.run(1)
    out = sol.state()
    sol.close()

    a = q.astype(np.float64)[:, 0, :] if axis == 0 else q.astype(np.float64)[:, :, 0]
    got = out[:, 0, :] if axis == 0 else out[:, :, 0]
    nm = 1 + axis
    vel = a[nm] / a[0]
    pr = (GAMMA - 1) * (a[3] - 0.5 * (a[1] ** 2 + a[2] ** 2) / a[0])
    f = a * vel
    f[nm] += pr
    f[3] += pr * vel
    ref = a - sign * dt * n * (f - np.roll(f, sign, axis=1))  # upstream differences
    weak = k == 1 if sign < 0 else k == 3  # its downstream cell is strong, its upstream cell weak
    for c in (0, nm, 3):
        assert (np.abs(got[c] - ref[c]) / np.abs(a[c]))[weak].max() <= 1e-6, c


@pytest.mark.parametrize("nx,ny,steps", [(70, 50, 6), (61, 517, 4), (1100, 700, 2)])
@pytest.mark.parametrize("wall", [0, 1])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_mirror_image(fv, prec, wall, nx, ny, steps):
    """A strong random state and its mirror images along each axis: the same
    bits mirrored, between walls too (there a face is its own mirror image, so
    its mass flux is exactly zero)."""
    rng = np.random.default_rng(nx)
    shape = (ny, nx)
    r, p = np.exp(rng.uniform(-1.5, 1.5, (2, *shape)))
    c = np.sqrt(GAMMA * p / r)
    q = conserved(r, 2 * c * rng.uniform(-1, 1, shape), 2 * c * rng.uniform(-1, 1, shape), p)

    def run(q):
        print(f"[euler faces] mirror {prec} wall {wall} {nx}x{ny}", flush=True)
        bc = fv.FV_BC_WALL if wall else fv.FV_BC_PERIODIC
        s = fv.Solver(q, prec=fv.FV_F64 if prec == "f64" else fv.FV_F32, bc_x=bc, bc_y=bc, lx=1.0, ly=ny / nx, cfl=0.3,
                      gamma=GAMMA)
        s.run(steps)
        t = s.time()
        out = s.state()
        s.close()
        return out, t

    def mirror(q, axis):
        o = (q[:, :, ::-1] if axis == 0 else q[:, ::-1, :]).copy()
        o[1 + axis] = -o[1 + axis]
        return o

    out, t = run(q)
    assert np.isfinite(out).all()
    for axis in (0, 1):
        img, t_img = run(mirror(q, axis))
        assert t_img == t
        assert np.array_equal(mirror(img, axis), out)
