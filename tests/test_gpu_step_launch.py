"""A Heun step in one launch: both stages of a tile in one workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 7), (59, 4), (60, 5), (61, 9), (62, 3 * 4), (64, 64), (121, 17), (130, 33),
                                   (61, 517), (121, 697)])
@pytest.mark.parametrize("wall", [(0, 0), (1, 1), (1, 0), (0, 1)])
@pytest.mark.parametrize("eqn,bed", [("swe", True), ("swe", False), ("euler", False)])
def test_same_bits_as_two_launches(eqn, bed, wall, nx, ny):
    """Six steps in one call (three pairs of single launches) against six
    calls of one step (two launches each), and five against five (an odd step
    at the end): the same cells, the same arithmetic, equal bits.  The last two
    sizes take tiles of 8 and of 12 rows, the others of 4."""
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
    print(f"[step launch] {eqn} bed={bed} wall={wall} {nx}x{ny}", flush=True)
    bc = [fv.FV_BC_WALL if w else fv.FV_BC_PERIODIC for w in wall]
    for steps in (6, 5):
        runs = []
        for calls in ([steps], [1] * steps):
            kw = dict(eqn=fv.FV_EULER) if eqn == "euler" else {}
            s = fv.Solver(q.astype(np.float32), None if b is None else b.astype(np.float32), prec=fv.FV_F32, bc_x=bc[0],
                          bc_y=bc[1], lx=1.0, ly=ny / nx, **kw)
            for k in calls:
                s.run(k)
            runs.append((s.state(), s.time()))
        assert np.isfinite(runs[0][0]).all()
        assert np.array_equal(runs[0][0], runs[1][0])
        assert runs[0][1] == runs[1][1]
