"""Learned, direct and blended steps on both sides of the split size, with a
network whose output matters."""
import numpy as np
import pytest

from parity import state_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["learned", "direct", "blend"])
@pytest.mark.parametrize("flux", ["hlle", "rusanov"])
@pytest.mark.parametrize("ny", [96, 104])
def test_periodic_copies_follow_the_network(scheme, flux, ny):
    """A solve of one round of 8 x 8 network tiles and the same data two by two
    (768 tiles, the last size in one launch per stage with HLLE, and 832): the
    same states.  The bound is 1e-2 of what the network's output is worth, the
    difference to the same solve with a zero last layer, and 1e-6 (twelve
    stages' FP32 rounding is below that)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    nx, steps = 128, 6
    rng = np.random.default_rng(5)
    layers = [(3, 32), (32, 32), (32, 32), (32, 32), (32, 72)]
    ws = [rng.standard_normal((co, ci, 3, 3)) * np.sqrt(2 / (9 * ci)) * (0.3 if co == 72 else 1) for ci, co in layers]
    bs = [rng.uniform(0, 0.1, co) for _, co in layers]
    none = ws[:-1] + [0 * ws[-1]], bs[:-1] + [0 * bs[-1]]
    y, x = np.mgrid[0:ny, 0:nx]
    a, b = 2 * np.pi * x / nx, 2 * np.pi * y / ny
    h = 1 + 0.1 * np.sin(8 * a) * np.cos(6 * b) + 0.05 * np.sin(3 * a + 5 * b)
    q = np.stack([h, 0.3 * h * np.cos(5 * b), 0.2 * h * np.sin(7 * a)]).astype(np.float32)

    def run(q, net):
        print(f"[learned split] {scheme} {flux} {q.shape}", flush=True)
        m = fv.Model(fv.params_to_vector(*net), fv.make_model_desc(mean=(1.0, 0.0, 0.0), inv_std=(5.0, 5.0, 5.0)))
        s = fv.Solver(q, prec=fv.FV_F32, dt_fixed=1e-3, learned=1, h_ref=1.0, lx=q.shape[2] / 64, ly=q.shape[1] / 64,
                      flux=fv.FV_FLUX_RUSANOV if flux == "rusanov" else fv.FV_FLUX_HLLE)
        stats = {"learned": s.learned_step, "direct": s.direct_step, "blend": s.blend_step}[scheme](m, steps)
        out = s.state()
        s.close()
        m.close()
        return out, stats

    (small, st), (small0, _) = run(q, (ws, bs)), run(q, none)
    big, st2 = run(np.tile(q, (1, 2, 2)), (ws, bs))
    worth = state_rel(small, small0)
    assert np.isfinite(big).all() and worth >= 1e-4, worth
    err = state_rel(big, np.tile(small, (1, 2, 2)))
    assert err <= min(1e-2 * worth, 1e-6), (err, worth)
    assert st2 == (4 * st[0], st[1])


@pytest.mark.parametrize("scheme", ["learned", "direct", "blend"])
@pytest.mark.parametrize("ny", [96, 104])
def test_redone_steps_on_both_sides(scheme, ny):
    """A shallow state and a large random head, so that steps fail and are
    redone with the plain scheme: the same decisions, counts and states two by
    two as alone (the redone step is the plain FP32 one: 1e-6)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from oracle import learned as L
    from paper_2602_08670_amd import fv
    from paper_2602_08670_amd import inputs as I

    nx, steps = 128, 3
    p = L.init_params(2, scale_last=10.0)
    vec = fv.params_to_vector([w.numpy() for w in p["w"]], [b.numpy() for b in p["b"]])
    q = I.random_smooth_swe(nx, seed=2)[:, :ny].astype(np.float32)
    q[0] *= 0.1

    def run(q):
        print(f"[learned split] redo {scheme} {q.shape}", flush=True)
        m = fv.Model(vec, fv.make_model_desc(mean=tuple(p["mean"].tolist()), inv_std=tuple(p["inv_std"].tolist())))
        s = fv.Solver(q, prec=fv.FV_F32, dt_fixed=2.5e-4, learned=1, h_ref=0.1, lx=q.shape[2] / nx, ly=q.shape[1] / nx)
        stats = {"learned": s.learned_step, "direct": s.direct_step, "blend": s.blend_step}[scheme](m, steps)
        out, t = s.state(), s.time()
        s.close()
        m.close()
        return out, stats, t

    small, st, t = run(np.ascontiguousarray(q))
    big, st2, t2 = run(np.tile(q, (1, 2, 2)))
    assert st[1] >= 1 and np.isfinite(small).all()
    assert st2 == (4 * st[0], st[1]) and t2 == t
    assert state_rel(big, np.tile(small, (1, 2, 2))) <= 1e-6
