"""GPU parity of the FP32 GEMMs' mirrored-offset steps and their parts with the
dense FP64 oracle, where they can go wrong: grids smaller and larger than a
tile, ragged depths, every form of the last bin chunk (whole, short, at most 2
bins), windows from zero to the full grid, more parts than a tile has steps, a
B-scan's parts over |d_x| and depth, and a window whose smallest chunk needs
more than 64 KiB of LDS."""
import numpy as np
import pytest

from oracle import operator as O
from paper_2012_04534_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL32 = 1e-5     # the FP32 operator's bound, norm-wise and element-wise


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def errs(got, ref):
    return max(np.linalg.norm(got - ref) / np.linalg.norm(ref), np.abs(got - ref).max() / np.abs(ref).max())


@pytest.mark.parametrize("nx,ny,nz,m,win,beam,adjoint", [
    (37, 1, 50, 19, -1, False, True),      # B-scan, ragged tile and depth, short last chunk
    (16, 1, 17, 16, 0, False, True),       # zero window, whole chunk
    (1, 1, 33, 5, -1, False, True),        # one position
    (300, 1, 9, 2, -1, False, False),      # forward wider than the LDS takes at 16 depths (adjoint refused:
                                           # its 300 delay rows of 64 depths alone exceed 64 KiB)
    (9, 6, 20, 18, -1, True, True),        # full C-scan with the beam, at most 2 last bins
    (5, 11, 48, 33, 2, False, True),       # narrow window, 1 last bin
    (21, 7, 16, 14, 3, True, True),        # several tiles in x, beam
    (190, 2, 8, 4, -1, False, False),      # forward chunk of 4 above 64 KiB of LDS (adjoint refused)
])
def test_mirrored_steps_and_parts(nx, ny, nz, m, win, beam, adjoint, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(nx, ny, nz, 512, win_x=win, win_y=win)
    if beam:
        g["theta"] = float(np.radians(25.0))
    bins, _ = u.ufss_select_freqs(g, m, False, 5 + m)
    A = O.dense_A(g, bins)
    x = W.cn((ny, nx, nz), 11).astype(np.complex64)
    r = W.cn((ny, nx, m), 12).astype(np.complex64)
    y_ref = (A @ x.reshape(-1).astype(np.complex128)).reshape(ny, nx, m)
    x_ref = (A.conj().T @ r.reshape(-1).astype(np.complex128)).reshape(ny, nx, nz)
    plan = u.Plan(g, m, False, bins, algo=u.ALGO_GEMM)
    xt, rt = torch.from_numpy(x).to(dev), torch.from_numpy(r).to(dev)
    yo, xo = torch.empty_like(rt), torch.empty_like(xt)
    # the default parts, one part, and more parts than steps (the widest window
    # takes 2 sub-tiles per wave only: 4 exceed the operator's window limit)
    ft = 4 if nx < 190 else 2
    for t in (None, dict(fwd_split=1, fwd_zsplit=1, adj_split=1),
              dict(fwd_split=64, fwd_zsplit=3, adj_split=64, fwd_tile=ft, adj_tile=4, fwd_chunk=8, adj_chunk=8),
              dict(fwd_split=7, fwd_zsplit=2, adj_split=5, fwd_tile=2, adj_tile=2, adj_waves=8)):
        if t:
            u.ufss_plan_set_tiling(plan, **t)
        u.ufss_forward(plan, xt, yo)
        assert errs(yo.cpu().numpy(), y_ref) < TOL32, t
        if adjoint:
            u.ufss_adjoint(plan, rt, xo)
            assert errs(xo.cpu().numpy(), x_ref) < TOL32, t
        else:
            with pytest.raises(u.UfssError) as e:
                u.ufss_adjoint(plan, rt, xo)
            assert e.value.name == "UNSUPPORTED"
    plan.close()
