"""K-cycles on pinned host vectors: the same bits as on device vectors, and the residual
crosses the bus once."""
import statistics
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1302_2547_amd import inputs  # noqa: E402


@pytest.fixture(scope="module")
def amg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1302_2547_amd import amg as mod
    return mod


def cliques(count, size):
    """CSR (device) of `count` cliques of `size` vertices in a row, the last vertex of each
    joined to the first of the next."""
    n = count * size
    k = torch.arange(n, device="cuda")
    first, last = (k % size == 0) & (k > 0), (k % size == size - 1) & (k < n - 1)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = (size + first.long() + last.long()).cumsum(0)
    col = torch.empty(int(rp[-1]), dtype=torch.int32, device="cuda")
    val = torch.full((int(rp[-1]),), -0.1, dtype=torch.float64, device="cuda")
    inside = ((rp[:-1] + first.long())[:, None] + torch.arange(size, device="cuda")).reshape(-1)
    col[inside] = ((k - k % size)[:, None] + torch.arange(size, device="cuda")).reshape(-1).int()
    val[inside] = -1.0
    val[rp[:-1] + first.long() + k % size] = size + 0.5
    col[rp[:-1][first]] = (k[first] - 1).int()
    col[rp[1:][last] - 1] = (k[last] + 1).int()
    return rp.int(), col, val


def median_us(call, reps=15):
    times = []
    for k in range(reps + 2):
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        times.append(1e6 * (time.perf_counter() - t))
    return statistics.median(times[2:])


def test_pinned_vectors_have_the_same_bits(amg):
    csr = [torch.from_numpy(v).cuda() for v in inputs.grid_laplacian((33, 31), jitter=0.1, seed=3)]
    with amg.Hierarchy(*csr) as h:
        r = torch.from_numpy(inputs.rhs(h.n, 4))
        want, z = torch.empty(h.n, dtype=torch.float64, device="cuda"), torch.empty(h.n, dtype=torch.float64, device="cuda")
        h.kcycle(r.cuda(), want)
        pr, pz = r.pin_memory(), torch.empty(h.n, dtype=torch.float64).pin_memory()
        h.kcycle(pr.data_ptr(), z)
        assert torch.equal(z, want)
        h.kcycle(pr.data_ptr(), pz.data_ptr())
        assert torch.equal(pz, want.cpu())
        h.kcycle(pr.data_ptr(), pr.data_ptr())  # in place
        assert torch.equal(pr, want.cpu())


# 300 entries a row: read in place by the two kernels that gather from it, the residual
# took 300 us more in pinned memory than on the device, where its copy takes 55.
def test_pinned_residual_costs_a_copy(amg):
    with amg.Hierarchy(*cliques(1000, 300), autotune=0) as h:
        r = torch.from_numpy(inputs.rhs(h.n, 4)).pin_memory()
        rd, z = r.cuda(), torch.empty(h.n, dtype=torch.float64, device="cuda")
        copy = median_us(lambda: rd.copy_(r))
        device = median_us(lambda: h.kcycle(rd, z))
        pinned = median_us(lambda: h.kcycle(r.data_ptr(), z))
    print(f"[pinned] copy {copy:.1f} us, K-cycle {device:.1f} us, from pinned memory {pinned:.1f} us", flush=True)
    assert pinned - device < 2.5 * copy
