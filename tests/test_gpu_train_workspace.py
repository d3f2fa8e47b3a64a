"""Trainers in less workspace than fv_train_workspace_bytes asks for."""
import numpy as np
import pytest

from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu


def al(n):
    return (n + 255) // 256 * 256


def least_bytes(B, nx, ny, T, euler):
    """Workspace without kept layer gradients: the rollout, one dz, two layer
    gradients, the rounded input and one pass's partial sums per 16 x 16 tile."""
    nv, cz = (4, 96) if euler else (3, 72)
    p = B * nx * ny
    st, act = al(p * nv * 4), al(p * 64)
    tiles = B * (nx // 16) * ((ny + 15) // 16)
    co = 16 * ((cz + 15) // 16)
    per_solve = 2 * al(B * 4) + 2 * al(B * 8) + al(B * 4) if not euler else al(B * 8) + 2 * al(B * 8) + al(B * 4)
    return ((T + 1) * st + T * st + T * 8 * act + T * 2 * al(p * cz * 4) + al(T * B * 4) + st + per_solve
            + al(p * 96 * 2) + al(p * 2 * 20 * 4 if not euler else p * 2 * ADJ_EULER * 4) + 3 * st
            + 2 * act + al(p * 32) + al(tiles * (9 * co * 32 + co) * 4) + al(1024 * 8) + 512)


ADJ_EULER = 24  # floats of a face's record of contributions


@pytest.mark.parametrize("euler", [False, True])
@pytest.mark.parametrize("B,nx,ny,T", [(1, 16, 8, 2), (3, 48, 20, 3), (16, 64, 64, 2)])
def test_less_workspace(B, nx, ny, T, euler):
    """All of it, half of what the kept layer gradients take, none of it: the
    same gradients (FP32 sums of the same terms in other orders: 1e-4 relative
    per layer), nothing written past the end; one byte less is refused."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    rng = np.random.default_rng(nx)
    nv, last = (4, 96) if euler else (3, 72)
    layers = [(nv, 32), (32, 32), (32, 32), (32, 32), (32, last)]
    ws = [rng.standard_normal((co, ci, 3, 3)) * np.sqrt(2 / (9 * ci)) * (0.05 if co == last else 1) for ci, co in layers]
    vec = fv.params_to_vector(ws, [rng.uniform(0, 0.05, co) for _, co in layers])
    n = max(nx, ny)
    gen = I.random_smooth_euler if euler else I.random_smooth_swe
    q0 = np.stack([gen(n, seed=s)[:, :ny, :nx] for s in range(B)])
    q0 = torch.tensor(np.ascontiguousarray(q0), dtype=torch.float32, device="cuda")
    tg = q0[None].repeat(T, 1, 1, 1, 1) + torch.tensor(rng.standard_normal((T, B, nv, ny, nx)) * 1e-3,
                                                     dtype=torch.float32, device="cuda")
    geo = dict(lx=nx / 64, ly=ny / 64)
    if euler:
        net = fv.EulerLearned(vec, B, nx, ny, 5e-4, **geo)
        cfg = fv.make_euler_train_config(B, nx, ny, T, 5e-4, **geo)
        full = fv.lib.fv_euler_train_workspace_bytes(cfg)
        create, step, destroy = fv.lib.fv_euler_train_create, fv.lib.fv_euler_train_step, fv.lib.fv_euler_train_destroy
    else:
        net = fv.Model(vec)
        cfg = fv.make_train_config(B, nx, ny, T, 5e-4, **geo)
        full = fv.lib.fv_train_workspace_bytes(cfg)
        create, step, destroy = fv.lib.fv_train_create, fv.lib.fv_train_step, fv.lib.fv_train_destroy
    import ctypes

    least = least_bytes(B, nx, ny, T, euler)
    assert least < full

    def run(nbytes):
        print(f"[train workspace] euler={euler} B={B} {nx}x{ny} T={T} {nbytes} of {full} bytes", flush=True)
        buf = torch.full((nbytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        g, m, v = torch.zeros(3, vec.size, dtype=torch.float32, device="cuda")
        h = ctypes.c_void_p()
        rc = create(ctypes.byref(cfg), net.h, g.data_ptr(), m.data_ptr(), v.data_ptr(), buf.data_ptr(), nbytes,
                    ctypes.byref(h))
        if rc != fv.FV_OK:
            return rc, None
        loss = ctypes.c_double()
        for _ in range(2):
            assert step(h, q0.data_ptr(), tg.data_ptr(), T, ctypes.byref(loss), None) == fv.FV_OK
        destroy(h)
        assert (buf[nbytes:] == 0x5A).all()
        return loss.value, g.double().cpu().numpy()

    loss, ref = run(full)
    assert np.isfinite(ref).all() and np.abs(ref).max() > 0
    for nbytes in (least, (least + full) // 512 * 256, full - 256):
        l2, g = run(nbytes)
        assert l2 == loss
        off = 0
        for ci, co in layers:
            k = co * ci * 9 + co
            assert np.linalg.norm(g[off:off + k] - ref[off:off + k]) <= 1e-4 * np.linalg.norm(ref[off:off + k])
            off += k
    assert run(least - 1) == (fv.FV_E_NOMEM, None)
