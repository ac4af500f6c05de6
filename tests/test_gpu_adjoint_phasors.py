"""The FP32 adjoint's phasor of a bin is that bin's own cosine and sine, whatever
its neighbours in the union: with measurements at one bin only, a union of
consecutive bins, one with a gap after them and one of every other bin give the
same bits, in the 4- and 8-wave kernels and in a batch.  (The 8-wave kernel on a
union of consecutive bins rotates phasors from one bin to the next; it is held to
the FP64 oracle's bound by the operator tests.)"""
import numpy as np
import pytest

from paper_2012_04534_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NX, NZ, N = 13, 70, 16


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def unions(slot, gap):
    """Two unions with the same bin at `slot`: consecutive bins, and every other
    bin; with `gap`, each followed by one more bin far off."""
    k0 = 60
    near = [k0 + i for i in range(N)]
    wide = [k0 + slot + 2 * (i - slot) for i in range(N)]
    return [np.array(b + ([120] if gap else []), dtype=np.int32) for b in (near, wide)]


def operand(ny, m, slot, dev):
    r = np.zeros((ny, NX, m), dtype=np.complex64)
    r[:, :, slot] = W.cn((ny, NX), 5)
    return torch.from_numpy(r).to(dev)


@pytest.mark.parametrize("waves,gap", [(4, False), (4, True), (8, True)])
@pytest.mark.parametrize("chunk,tile", [(16, 2), (16, 4), (8, 2)])
@pytest.mark.parametrize("ny", [1, 9])
def test_phasors_do_not_depend_on_the_neighbouring_bins(waves, gap, chunk, tile, ny, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(NX, ny, NZ, 512)
    for slot in (1, 6, 11, 15):
        out = []
        for bins in unions(slot, gap):
            plan = u.Plan(g, len(bins), False, bins, algo=u.ALGO_GEMM)
            u.ufss_plan_set_tiling(plan, adj_waves=waves, adj_chunk=chunk, adj_tile=tile)
            x = torch.empty((ny, NX, NZ), dtype=torch.complex64, device=dev)
            u.ufss_adjoint(plan, operand(ny, len(bins), slot, dev), x)
            out.append(x)
            plan.close()
        assert torch.equal(out[0], out[1]), slot


@pytest.mark.parametrize("ny", [1, 9])
def test_phasors_of_a_batch(ny, dev):
    from paper_2012_04534_amd import ufss as u
    g = W.geometry(NX, ny, NZ, 512)
    for slot in (1, 6, 11, 15):
        xs = [torch.zeros((ny, NX, NZ), dtype=torch.complex64, device=dev) for _ in range(2)]
        bins = unions(slot, False)
        plans = [u.Plan(g, N, False, b, algo=u.ALGO_GEMM) for b in bins]
        batch = u.Batch(plans, [operand(ny, N, slot, dev)] * 2, xs, [1e-6] * 2, [1.0] * 2, 1)
        batch.run()                       # x = soft(A^H y, 1e-6)
        assert torch.equal(xs[0], xs[1]), slot
        assert float(xs[0].abs().max()) > 0
        batch.close()
        for p in plans:
            p.close()
