"""Learned, direct and blended steps past three rounds of 8 x 8 tiles: the
network pass and the stage as separate launches."""
import numpy as np
import pytest

from parity import state_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["learned", "direct", "blend"])
@pytest.mark.parametrize("nx,ny", [(128, 96), (128, 104)])
def test_periodic_copies(scheme, nx, ny):
    """A solve of one round of tiles and the same data two by two (768 tiles,
    the last size in one launch per stage, and 832): the same states, to the
    rounding of four steps in FP32 (below 1e-6; 1e-5)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    rng = np.random.default_rng(5)
    layers = [(3, 32), (32, 32), (32, 32), (32, 32), (32, 72)]
    ws = [rng.standard_normal((co, ci, 3, 3)) * np.sqrt(2 / (9 * ci)) * (0.02 if co == 72 else 1) for ci, co in layers]
    vec = fv.params_to_vector(ws, [rng.uniform(0, 0.02, co) for _, co in layers])
    y, x = np.mgrid[0:ny, 0:nx]
    h = 1 + 0.05 * np.sin(2 * np.pi * x / nx) * np.cos(2 * np.pi * y / ny)
    q = np.stack([h, 0.02 * h * np.cos(2 * np.pi * y / ny), 0.02 * h * np.sin(2 * np.pi * x / nx)]).astype(np.float32)

    def run(q):
        print(f"[routes] {scheme} {q.shape}", flush=True)
        m = fv.Model(vec)
        s = fv.Solver(q, prec=fv.FV_F32, dt_fixed=5e-4, learned=1, h_ref=1.0, lx=q.shape[2] / 64, ly=q.shape[1] / 64)
        {"learned": s.learned_step, "direct": s.direct_step, "blend": s.blend_step}[scheme](m, 4)
        out = s.state()
        s.close()
        m.close()
        return out

    small, big = run(q), run(np.tile(q, (1, 2, 2)))
    assert np.isfinite(big).all()
    assert state_rel(big, np.tile(small, (1, 2, 2))) <= 1e-5
