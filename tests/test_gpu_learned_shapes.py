"""GPU parity of the learned network's convolution kernels with the FP64 oracle
at the shapes where their runs change: fewer columns than a run, remainders,
one row or one depth, one to eight channels, and a grid of several
weight-gradient ranges.  Forward against the oracle network, gradients of the
last stage's weights against central differences of the oracle loss."""
import numpy as np
import pytest

from oracle import learned as N
from oracle import operator as O
from oracle import solver as V
from paper_2012_04534_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,ch", [(1, 1, 20, 1), (2, 3, 7, 5), (3, 1, 16, 8), (5, 2, 1, 8), (7, 4, 9, 7),
                                         (6, 5, 300, 2)])
def test_shapes(nx, ny, nz, ch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_04534_amd import ufss as u
    dev, S, shape, m = torch.device("cuda:0"), 2, (ny, nx, nz), 4
    g = W.geometry(nx, ny, nz, 64, win_x=1, win_y=1)
    bins, _ = u.ufss_select_freqs(g, m, False, 3)
    Am = O.dense_A(g, bins)
    A, AH = (lambda v: Am @ v), (lambda v: Am.conj().T @ v)
    y = W.cn((ny, nx, m), 5).astype(np.complex64)
    L = 1.01 * V.lipschitz_dense(Am)
    plan = u.Plan(g, m, False, bins, algo=u.ALGO_GEMM)
    net = u.Net(plan, stages=S, channels=ch, L=L, mu=0.1)
    n = N.stage_size(ch)
    rng = np.random.default_rng(8)
    p = (0.05 * rng.standard_normal(S * n)).astype(np.float32)
    u.ufss_unrolled_params(net, set_to=p)
    yt = torch.from_numpy(y).to(dev)
    x = torch.zeros(shape, dtype=torch.complex64, device=dev)
    u.ufss_unrolled_forward(net, yt, x)
    yd, pd = y.reshape(-1).astype(np.complex128), p.astype(np.float64)
    xo = N.forward(A, AH, yd, pd, S, ch, L, 0.1, shape)
    assert np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo) < 1e-5
    a_ref = (0.5 * W.cn(shape, 13)).astype(np.complex64)
    _, grad = u.ufss_unrolled_grad(net, yt, torch.from_numpy(a_ref).to(dev))
    b = (S - 1) * n
    idx = [b, b + 1] + list(b + 2 + rng.choice(ch * 54, 6, replace=False)) + [b + 2 + ch * 54 + ch - 1]
    idx += list(b + 2 + ch * 55 + rng.choice(ch * 54, 6, replace=False)) + [b + n - 2, b + n - 1]
    # step 1e-5: the loss is near 1 and the gradients as small as 1e-8, so a step of
    # 1e-6 leaves the rounding of the two losses (2^-53 / 1e-6 = 1e-10) in the
    # result, and 1e-4 moves a unit across its ReLU's kink
    fd = N.fd_grad(A, AH, yd, pd, S, ch, L, 0.1, shape, a_ref.astype(np.complex128), idx, h=1e-5)
    assert np.linalg.norm(grad[idx] - fd) / np.linalg.norm(fd) < 1e-3
    net.close()
    plan.close()


@pytest.mark.parametrize("nx,ny,nz", [(2, 17, 18), (5, 64, 3), (3, 65, 2), (20, 1, 33)])
def test_transform_plan_shapes(nx, ny, nz):
    """The proximal step in the transform path's last product: tiles of rows, the most
    rows of one column and one more (a pass of its own), against the oracle network."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_04534_amd import ufss as u
    dev, S, ch, shape, m = torch.device("cuda:0"), 2, 3, (ny, nx, nz), 4
    g = W.geometry(nx, ny, nz, 64, win_x=1, win_y=1)
    bins, _ = u.ufss_select_freqs(g, m, False, 3)
    Am = O.dense_A(g, bins)
    y = W.cn((ny, nx, m), 5).astype(np.complex64)
    plan = u.Plan(g, m, False, bins, algo=u.ALGO_FFT)
    L = u.ufss_lipschitz(plan)
    net = u.Net(plan, stages=S, channels=ch, L=L, mu=0.1)
    p = (0.05 * np.random.default_rng(8).standard_normal(S * N.stage_size(ch))).astype(np.float32)
    u.ufss_unrolled_params(net, set_to=p)
    x = torch.zeros(shape, dtype=torch.complex64, device=dev)
    u.ufss_unrolled_forward(net, torch.from_numpy(y).to(dev), x)
    xo = N.forward(lambda v: Am @ v, lambda v: Am.conj().T @ v, y.reshape(-1).astype(np.complex128),
                   p.astype(np.float64), S, ch, L, 0.1, shape)
    assert np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo) < 1e-5
    net.close()
    plan.close()
