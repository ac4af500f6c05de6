"""The FP32 GEMMs on a scene: point scatterers over a back wall, whose measurements
add up at a few voxels and cancel at the others.  One product for mirrored offsets
may round no worse there than a plain FP32 sum over the window, offset by offset and
row by row, each row's sum added to the whole (torch, the phasors rounded from FP64;
the same sum in FP64, which the oracle checks at a few places, is the reference)."""
import numpy as np
import pytest

from oracle import geometry as G
from oracle import operator as O
from paper_2012_04534_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def shifted(v, dy, dx):
    """v[p + d] on the grid [ny, nx, ...], zero outside."""
    ny, nx = v.shape[:2]
    out = torch.zeros_like(v)
    out[max(0, -dy):min(ny, ny - dy), max(0, -dx):min(nx, nx - dx)] = \
        v[max(0, dy):min(ny, ny + dy), max(0, dx):min(nx, nx + dx)]
    return out


def plain(g, bins, v, adjoint, dtype, dev):
    """A (unit spectrum) or its adjoint on [ny, nx, .], summed in dtype."""
    wx, wy = G.window(g)
    nz = g["nz"]
    n = nz if adjoint else len(bins)
    re, im = (torch.from_numpy(np.ascontiguousarray(a)).to(dev, dtype) for a in (v.real, v.imag))
    total = [torch.zeros(v.shape[:2] + (n,), dtype=dtype, device=dev) for _ in range(2)]
    for dy in range(-wy, wy + 1):
        row = [torch.zeros_like(t) for t in total]
        for dx in range(-wx, wx + 1):
            # A's entries at this offset, unit modulus: [m, nz]
            e = O.entries(g, bins, abs(dx), abs(dy), np.zeros(nz, int), np.zeros(nz, int), np.arange(nz), True)
            e = e.conj() if adjoint else e.T
            c, s = (torch.from_numpy(np.ascontiguousarray(a)).to(dev, dtype) for a in (e.real, e.imag))
            a, b = shifted(re, dy, dx), shifted(im, dy, dx)
            for j in range(v.shape[2]):
                aj, bj = a[:, :, j, None], b[:, :, j, None]
                row[0] += aj * c[j]
                row[0] -= bj * s[j]
                row[1] += aj * s[j]
                row[1] += bj * c[j]
        for t, r in zip(total, row):
            t += r
    return (total[0].double() + 1j * total[1].double()).cpu().numpy()


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("nx,ny,nz,m,win", [(24, 28, 16, 12, 16), (18, 19, 20, 14, -1)])
def test_scene_rounds_no_worse_than_a_plain_sum(nx, ny, nz, m, win, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(nx, ny, nz, 128, win_x=win, win_y=win)
    bins, _ = u.ufss_select_freqs(g, m, False, 3)
    h = G.pulse_spectrum(g, bins)
    x = W.scene(g, 12, seed=4).astype(np.complex64)
    x[:, :, nz - 6] = 1.0
    y = (plain(g, bins, x, False, torch.float64, dev) * h).astype(np.complex64)
    hy = (y * h.astype(np.float32)).astype(np.complex64)             # the adjoint's operand
    a_ref = plain(g, bins, hy, True, torch.float64, dev)
    image = a_ref.astype(np.complex64)
    y_ref = plain(g, bins, image, False, torch.float64, dev) * h
    for py, px in ((0, 0), (ny // 2, nx - 2)):
        assert rel(y_ref[py, px], O.apply_A_at(g, bins, image, py, px)) < 1e-10
        assert rel(a_ref[py, px], O.apply_AH_at(g, bins, y, py, px)) < 1e-6        # h rounded to FP32

    plan = u.Plan(g, m, False, bins, algo=u.ALGO_GEMM)
    at, yt = (torch.empty((ny, nx, n), dtype=torch.complex64, device=dev) for n in (nz, m))
    u.ufss_adjoint(plan, torch.from_numpy(y).to(dev), at)
    u.ufss_forward(plan, torch.from_numpy(image).to(dev), yt)
    assert rel(at.cpu().numpy(), a_ref) <= rel(plain(g, bins, hy, True, torch.float32, dev), a_ref)
    assert rel(yt.cpu().numpy(), y_ref) <= rel(plain(g, bins, image, False, torch.float32, dev) * h, y_ref)
    plan.close()
