"""Stage kernels on rows of tens of millions of cells."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_offsets_within_a_tile():
    """36 million columns by 16 rows in double precision (13.8 GB of state):
    sixteen such rows are more than 4 GiB, eight are not.  Data of period 64
    along x, the same in every row, two steps: every row and every period is
    the small grid's, bit for bit."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    from paper_2602_08670_amd import fv

    nx, ny, p = 36_000_000, 16, 64
    x = 2 * np.pi * np.arange(p) / p
    h = 1 + 0.1 * np.sin(x)
    one = np.stack([h, 0.3 * h * np.cos(x), 0.1 * h])
    kw = dict(prec=fv.FV_F64, dt_fixed=1e-3, h_ref=1.0)
    s = fv.Solver(np.repeat(one[:, None, :], ny, axis=1), lx=p / 64, ly=ny / 64, **kw)
    s.run(2)
    ref = s.state()
    s.close()
    assert (ref == ref[:, :1]).all() and np.abs(ref[:, 0] - one).max() > 0

    print(f"[long rows] {nx} x {ny}", flush=True)
    cfg = fv.make_config(nx=nx, ny=ny, eqn=fv.FV_SWE, lx=nx / 64, ly=ny / 64, **kw)
    q = torch.empty((3, ny, nx // p, p), dtype=torch.float64, device="cuda")
    q[:] = torch.tensor(one, device="cuda")[:, None, None, :]
    n = fv.fv_workspace_bytes(cfg)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    handle = fv.fv_init(cfg, q.data_ptr(), None, ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    fv.fv_run(handle, 2)
    assert fv.fv_time(handle)[1] == 2
    want = torch.tensor(ref[:, 0], device="cuda")
    same = all(bool((q[v, y] == want[v]).all()) for v in range(3) for y in range(ny))
    fv.fv_destroy(handle)
    del q, ws
    torch.cuda.empty_cache()
    assert same
