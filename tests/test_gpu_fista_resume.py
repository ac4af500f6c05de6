"""FISTA stopped and resumed through (x, gamma, k_done) gives the iterates and
residuals of one uninterrupted call bit for bit, on every operator path: the
transform path with its fused passes (one to four tiles of rows, FP32 and BF16
tables, equal and unequal axes), the same path with a kernel per pass (more than
64 rows), and the GEMM and phasor paths."""
import numpy as np
import pytest

from paper_2012_04534_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("algo,bf16,nx,ny,nz,m,per,win,real,accel", [
    ("fft", False, 17, 17, 50, 11, True, -1, False, True),    # equal axes, two tiles of rows
    ("fft", True, 9, 16, 65, 33, True, -1, False, True),      # unequal axes, one tile, BF16 table
    ("fft", True, 33, 33, 21, 6, False, 5, False, True),      # equal axes, three tiles, BF16 table
    ("fft", False, 10, 64, 9, 20, True, 3, True, True),       # four tiles, real reflectivity
    ("fft", False, 40, 1, 60, 8, False, -1, False, False),    # B-scan, ISTA
    ("fft", False, 9, 65, 7, 20, True, 3, False, True),       # a kernel per pass
    ("gemm", False, 20, 13, 40, 17, True, 4, False, True),
    ("gemm", True, 20, 13, 40, 17, True, 4, False, True),
    ("phasor", False, 12, 10, 30, 2, True, -1, False, True),
])
def test_resumed_run_is_bitwise_the_uninterrupted_one(algo, bf16, nx, ny, nz, m, per, win, real, accel, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(nx, ny, nz, 1024, win_x=win, win_y=win)
    bins, _ = u.ufss_select_freqs(g, m, per, 7 + m)
    plan = u.Plan(g, m, per, bins, dtype=u.BF16 if bf16 else u.F32,
                  algo={"fft": u.ALGO_FFT, "gemm": u.ALGO_GEMM, "phasor": u.ALGO_PHASOR}[algo])
    L = u.ufss_lipschitz(plan)
    shape = (ny, nx, nz)
    y = torch.empty((ny, nx, m), dtype=torch.complex64, device=dev)
    u.ufss_forward(plan, torch.from_numpy((W.cn(shape, 3) * (np.arange(nz) % 7 == 0)).astype(np.complex64)).to(dev), y)
    x0 = torch.from_numpy((0.01 * W.cn(shape, 4)).astype(np.complex64)).to(dev)
    g0 = torch.empty(shape, dtype=torch.complex64, device=dev)
    u.ufss_adjoint(plan, y, g0)
    lam = 0.02 * u.ufss_absmax(g0)

    def run(parts):
        x = x0.clone()
        state, res = {"gamma": torch.zeros_like(x), "k_done": 0}, []
        for n in parts:
            res.append(u.ufss_fista(plan, y, lam, L, n, x, accel=accel, state=state, real=real)["res"])
        assert state["k_done"] == sum(parts)
        return x, state["gamma"], np.concatenate(res)

    x, gamma, res = run([7])
    assert np.linalg.norm(x.cpu().numpy()) > 0
    for parts in ([3, 4], [1, 1, 5]):
        xs, gs, rs = run(parts)
        assert torch.equal(xs, x) and torch.equal(gs, gamma), parts
        assert np.array_equal(rs, res), parts
    plan.close()
