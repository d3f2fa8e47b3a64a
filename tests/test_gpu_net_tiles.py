"""The network pass on wide tiles with its weights in registers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("euler", [False, True])
@pytest.mark.parametrize("B,nx,ny", [
    (300, 16, 8),     # one tile per solve, rows and columns wrapping onto themselves
    (130, 48, 20),    # the last tile row overlaps the one before
    (70, 80, 40),     # the widest tile that spans a row
    (10, 96, 72),     # tiles within a row, a margin on each side
    (3, 112, 136),    # the last tile column overlaps the one before
    (40, 128, 128),   # several rounds of tiles
])
def test_same_bits_as_small_tiles(B, nx, ny, euler):
    """The same MFMAs per output in the same order as the pass on 8 x 8 tiles:
    equal bits.  Sides that 8 does not divide are compared on the grid stacked
    twice (rows of a periodic grid)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    rng = np.random.default_rng(nx + ny)
    nv, last = (4, 96) if euler else (3, 72)
    layers = [(nv, 32), (32, 32), (32, 32), (32, 32), (32, last)]
    vec = fv.params_to_vector([rng.standard_normal((co, ci, 3, 3)) * np.sqrt(2 / (9 * ci)) for ci, co in layers],
                              [rng.uniform(-0.1, 0.1, co) for _, co in layers])
    q = torch.tensor(rng.uniform(0.8, 1.2, (B, nv, ny, nx)), dtype=torch.float32, device="cuda")
    rep = 1 if ny % 8 == 0 else 2
    qq = q.repeat(1, 1, rep, 1)
    print(f"[net tiles] euler={euler} B={B} {nx}x{ny}", flush=True)
    if euler:
        a = fv.EulerLearned(vec, B, nx, ny, 1e-4, lx=nx / 64, ly=ny / 64).forward(q)
        b = fv.EulerLearned(vec, B, nx, rep * ny, 1e-4, lx=nx / 64, ly=rep * ny / 64).forward_tiled(qq)
    else:
        m = fv.Model(vec)
        a, b = m.forward(q), m.forward_tiled(qq)
    torch.cuda.synchronize()
    assert torch.isfinite(a).all()
    assert torch.equal(a, b[:, :ny])
