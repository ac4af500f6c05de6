"""FISTA's fused passes (forward post + adjoint pre, the update between the transform
path's products, statistics reduced one iteration late) against the same
iterations from the operator calls and an FP64 update: one to eight lanes per
sum, union rows with unselected bins, BF16 operands, odd sizes, one position,
and a grid with more blocks of partials than the fused update has room for."""
import numpy as np
import pytest

from oracle import solver as V
from paper_2012_04534_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# The operands of A and A^H are the same bits; an FP32 update is within 4 roundings
# (2.4e-7) of the FP64 one, three times over momentum 1 + 2 beta <= 3 in 3 iterations.
TOL32 = 2e-6
# A difference of 1e-7 moves one BF16 rounding (2^-8) in 2e4: sqrt(5e-5) 4e-3.
TOL16 = 1e-4


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("algo,bf16,nx,ny,nz,m,per,win,real,ref,iters", [
    ("gemm", False, 32, 1, 40, 20, False, -1, False, True, 3),
    ("gemm", False, 33, 9, 64, 40, True, -1, False, False, 3),     # many parts: several lanes per sum
    ("gemm", False, 12, 11, 30, 3, True, 1, True, True, 2),
    ("gemm", True, 20, 13, 40, 17, True, 4, False, True, 3),
    ("gemm", True, 24, 1, 33, 9, False, -1, False, False, 1),
    ("fft", False, 17, 17, 50, 11, True, -1, False, True, 3),
    ("fft", False, 19, 6, 31, 5, False, 3, True, False, 3),
    ("fft", True, 9, 16, 65, 33, True, -1, False, True, 3),
    ("fft", False, 1, 1, 12, 3, False, -1, False, True, 3),
    ("fft", False, 130, 2, 7, 2, True, 4, False, False, 2),        # more than one block of rows
    ("fft", False, 1024, 1, 832, 2, False, 0, False, True, 2),     # partials past the fused update's room
    ("fft", False, 150, 100, 5, 2, True, 1, False, True, 3),       # more than 64 rows: a kernel per product
    ("fft", False, 10, 64, 6, 20, True, 3, False, True, 3),        # the most rows of one column
    ("fft", False, 9, 65, 6, 20, True, 3, False, False, 3),        # one more
    ("fft", False, 5, 47, 20, 19, False, -1, True, True, 2),       # three tiles of rows
    ("fft", False, 16, 16, 17, 40, True, -1, True, True, 3),       # exactly one tile per axis
    ("fft", True, 40, 33, 9, 3, True, 5, False, False, 2),         # several tiles, transforms past one staged run
])
def test_fista_matches_the_operator_calls(algo, bf16, nx, ny, nz, m, per, win, real, ref, iters, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(nx, ny, nz, 1024, win_x=win, win_y=win)
    bins, _ = u.ufss_select_freqs(g, m, per, 5 + m)
    plan = u.Plan(g, m, per, bins, dtype=u.BF16 if bf16 else u.F32, algo=u.ALGO_FFT if algo == "fft" else u.ALGO_GEMM)
    L = u.ufss_lipschitz(plan)
    A = lambda x: call(u.ufss_forward, x, (ny, nx, m))
    AH = lambda r: call(u.ufss_adjoint, r, (ny, nx, nz))

    def call(fn, v, shape):
        out = torch.empty(shape, dtype=torch.complex64, device=dev)
        fn(plan, torch.from_numpy(np.ascontiguousarray(v).astype(np.complex64)).to(dev), out)
        return out.cpu().numpy().astype(np.complex128)

    x0 = W.cn((ny, nx, nz), 31)
    if real:
        x0 = x0.real + 0j
    y = A(x0 * (np.arange(nz) % 5 == 0)).astype(np.complex64)
    aref = (x0 + 0.1 * W.cn(x0.shape, 32)).astype(np.complex64) if ref else None
    lam = 0.05 * np.abs(AH(y)).max()
    xt = torch.zeros((ny, nx, nz), dtype=torch.complex64, device=dev)
    got = u.ufss_fista(plan, torch.from_numpy(y).to(dev), lam, L, iters, xt, real=real,
                       a_ref=None if aref is None else torch.from_numpy(aref).to(dev))
    a = gam = np.zeros((ny, nx, nz), dtype=np.complex64)
    t, tol, yn = 1.0, TOL16 if bf16 else TOL32, np.linalg.norm(y)
    for k in range(iters):
        r = (A(gam).astype(np.complex64) - y).astype(np.complex128)
        g1 = np.abs(gam.astype(np.complex128)).sum()
        res = np.linalg.norm(r)
        assert abs(got["res"][k] - res) < tol * yn
        assert abs(got["obj"][k] - (0.5 * res ** 2 + lam * g1)) < tol * (yn ** 2 + lam * g1)
        z = gam - AH(r) / L
        new = V.soft(z.real + 0j if real else z, lam / L)
        tn = 0.5 * (1.0 + np.sqrt(1.0 + 4.0 * t * t))
        gam = (new + (t - 1.0) / tn * (new - a.astype(np.complex128))).astype(np.complex64)
        change = np.linalg.norm(new - a) / np.linalg.norm(new)
        assert abs(got["rel_change"][k] - change) < 4 * tol
        if ref:
            assert abs(got["err_ref"][k] - np.linalg.norm(new - aref) / np.linalg.norm(aref)) < 4 * tol
        a, t = new.astype(np.complex64), tn
    assert np.linalg.norm(xt.cpu().numpy() - a) < tol * np.linalg.norm(a)
    plan.close()
