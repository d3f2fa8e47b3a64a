"""Face adjoints of training, 128 cells of the batch to a workgroup."""
import numpy as np
import pytest

from paper_2602_08670_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["learned", "blend", "direct"])
@pytest.mark.parametrize("B,nx,ny", [(2, 16, 4), (2, 16, 12), (4, 48, 20)])
def test_batch_gradient_is_the_mean_of_its_solves(scheme, B, nx, ny):
    """Half a workgroup's cells per solve, workgroups across two solves and one
    cut short: the batch's gradient equals the mean of its solves' own, which
    start their workgroups at their own first cell: FP32 sums of the same terms
    in different orders (B is a power of two, so that the loss scale does not
    change a bfloat16 rounding), 1e-4 relative per layer."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2602_08670_amd import fv

    rng = np.random.default_rng(B)
    layers = [(3, 32), (32, 32), (32, 32), (32, 32), (32, 72)]
    ws = [rng.standard_normal((co, ci, 3, 3)) * np.sqrt(2 / (9 * ci)) * (0.05 if co == 72 else 1) for ci, co in layers]
    vec = fv.params_to_vector(ws, [rng.uniform(0, 0.05, co) for _, co in layers])
    n = max(nx, ny)
    q0 = np.stack([I.random_smooth_swe(n, seed=s)[:, :ny, :nx] for s in range(B)])
    q0 = torch.tensor(np.ascontiguousarray(q0), dtype=torch.float32, device="cuda")
    tg = q0[None] + torch.tensor(rng.standard_normal((1, *q0.shape)) * 1e-3, dtype=torch.float32, device="cuda")
    print(f"[adjoint tiles] {scheme} B={B} {nx}x{ny}", flush=True)

    def grads(q, t):
        m = fv.Model(vec)
        kw = {"direct": dict(direct=1), "blend": dict(blend=1)}.get(scheme, {})
        tr = fv.Trainer(m, fv.make_train_config(q.shape[0], nx, ny, 1, 5e-4, lx=nx / 64, ly=ny / 64, **kw))
        tr.step(q.contiguous(), t.contiguous())
        g = tr.grads.double().cpu().numpy()
        tr.close()
        m.close()
        return g

    whole = grads(q0, tg)
    parts = np.mean([grads(q0[b:b + 1], tg[:, b:b + 1]) for b in range(B)], axis=0)
    assert np.isfinite(whole).all() and np.abs(parts).max() > 0
    off = 0
    for ci, co in layers:
        k = co * ci * 9 + co
        assert np.linalg.norm(whole[off:off + k] - parts[off:off + k]) <= 1e-4 * np.linalg.norm(parts[off:off + k])
        off += k
