"""The transform path keeps FP32's precision for inputs near the lower end of its
range, also where the table is BF16: scaling an input by a power of two scales the
result.  At 2^-120 an operand of order one holds digits down to 2^-149, so its own
rounding is 2^-30 of it; two FP32 roundings of the result (2^-22) bound the rest."""
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


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("nx,ny,nz,m", [
    (12, 12, 40, 9),        # equal axes: up to 8 members, three planes
    (12, 9, 40, 9),         # unequal axes: up to 4 members, two planes
    (6, 6, 600, 300),       # several staged chunks each way
    (7, 5, 600, 300),
])
def test_small_inputs_keep_their_digits(bf16, nx, ny, nz, m, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(nx, ny, nz, 4096 if m > 100 else 256)
    bins, _ = u.ufss_select_freqs(g, m, False, 1)
    plan = u.Plan(g, m, False, bins, dtype=u.BF16 if bf16 else u.F32, algo=u.ALGO_FFT)
    x = W.cn((ny, nx, nz), 1).astype(np.complex64)
    r = W.cn((ny, nx, m), 2).astype(np.complex64)

    def both(sx, sr):
        y = torch.empty((ny, nx, m), dtype=torch.complex64, device=dev)
        a = torch.empty((ny, nx, nz), dtype=torch.complex64, device=dev)
        u.ufss_forward(plan, torch.from_numpy((x * sx).astype(np.complex64)).to(dev), y)
        u.ufss_adjoint(plan, torch.from_numpy((r * sr).astype(np.complex64)).to(dev), a)
        return [t.cpu().numpy().astype(np.complex128) for t in (y, a)]

    def err(got, want):
        return np.linalg.norm(got - want) / np.linalg.norm(want)

    want = both(1.0, 1.0)
    for e in (60, 108, 112, 116, 120):
        for got, ref in zip(both(np.float32(2.0 ** -e), np.float32(2.0 ** -e)), want):
            assert err(got * 2.0 ** e, ref) < 2.0 ** -22, e
    # one depth (bin) of order one among small ones, in each position of the staged chunks
    for at in (0, 255, 256, 511):
        if at >= nz or at >= m:
            continue
        sx, sr = np.full(nz, 2.0 ** -112, np.float32), np.full(m, 2.0 ** -112, np.float32)
        sx[at] = sr[at] = 1.0
        only_x, only_r = np.zeros(nz, np.float32), np.zeros(m, np.float32)
        only_x[at] = only_r[at] = 1.0
        for got, ref in zip(both(sx, sr), both(only_x, only_r)):
            assert err(got, ref) < 2.0 ** -22, at
    # a first chunk of zeros, or of values of order one, before small ones
    if min(nz, m) > 256:
        zx, zr = (np.full(n, 2.0 ** -120, np.float32) for n in (nz, m))
        zx[:256] = zr[:256] = 0.0
        ox, orr = ((v > 0).astype(np.float32) for v in (zx, zr))
        for got, ref in zip(both(zx, zr), both(ox, orr)):
            assert err(got * 2.0 ** 120, ref) < 2.0 ** -22
    plan.close()
