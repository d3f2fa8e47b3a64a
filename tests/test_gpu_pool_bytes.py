"""Device memory that nothing uses is not asked for."""
import ctypes

import numpy as np
import pytest

from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fv():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv as F

    return F


def test_pool_of_one_learned_solve(fv):
    """A pool of the server's lists and one learned solve's buffers serves that
    solve: with a model, by default, no part of the pool is set aside."""
    rng = np.random.default_rng(3)
    m = fv.Model((rng.standard_normal(fv.fv_model_param_count()) * 0.02).astype(np.float32))
    q = I.random_smooth_swe(64, seed=1).astype(np.float32)
    kw = dict(max_solves=2, steps_per_round=4, max_items=1 << 12)
    ov = fv.lib.fv_server_pool_overhead(fv.fv_server_config(ctypes.sizeof(fv.fv_server_config), 2, 4, 0, 1 << 12))
    one = fv.Server.request_bytes(fv.make_request(q, 5, learned=True, dt_fixed=5e-4)[0])
    print(f"[pool bytes] overhead {ov}, solve {one}", flush=True)
    srv = fv.Server(ov + one, model=m, **kw)
    rid = srv.submit(q, 5, learned=True, dt_fixed=5e-4)
    rounds = 0
    while srv.round() != (0, 0):
        rounds += 1
        assert rounds < 10
    inf = srv.info(rid)
    out = srv.result(rid, q.shape)
    srv.close()
    assert inf.state == 2 and inf.steps_done == 5
    s = fv.Solver(q, prec=fv.FV_F32, dt_fixed=5e-4, learned=1)
    s.learned_step(m, 5)
    assert np.array_equal(out, s.state().astype(np.float32))


@pytest.mark.parametrize("B,nx,ny", [(64, 64, 64), (2, 32, 4), (3, 16, 8)])
def test_forward_scratch(fv, B, nx, ny):
    """A forward allocates its output and the scratch that its shape uses: two
    activation planes of 64 bytes per cell below eight rows, none from there
    on; z is the one-launch pass's where that takes the shape."""
    import torch

    rng = np.random.default_rng(5)
    m = fv.Model((rng.standard_normal(fv.fv_model_param_count()) * 0.02).astype(np.float32))
    q = torch.tensor(rng.uniform(0.8, 1.2, (B, 3, ny, nx)), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    z = m.forward(q)
    torch.cuda.synchronize()
    extra = torch.cuda.max_memory_allocated() - before - z.numel() * 4
    print(f"[pool bytes] forward {B} x {nx}x{ny}: {extra} bytes", flush=True)
    assert extra <= (1024 if ny >= 8 else 2 * 64 * B * nx * ny + 1024)
    assert torch.isfinite(z).all()
    if ny >= 8:
        assert torch.equal(z, m.forward_tiled(q))
