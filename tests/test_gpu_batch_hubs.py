"""Post-smoothing of a batch in two launches on a mid-size level with hub rows: a column
has the bits that it has alone, where one launch smooths it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sp = pytest.importorskip("scipy.sparse")

import oracle  # noqa: E402
from paper_1302_2547_amd import inputs  # noqa: E402


@pytest.fixture(scope="module")
def amg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1302_2547_amd import amg as mod
    return mod


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def hubs_in_a_grid(side, spokes):
    """A 3D grid with a vertex joined to spokes[k] others for every k: a hub takes its
    neighbours, and theirs are its neighbours on level 1."""
    rp, ci, va = inputs.grid_laplacian((side,) * 3, jitter=0.1, seed=9)
    n = len(rp) - 1
    a = sp.csr_matrix((va, ci, rp), shape=(n, n))
    rng = np.random.default_rng(5)
    for k, count in enumerate(spokes):
        to = rng.choice(n // len(spokes), count, replace=False) + k * (n // len(spokes))
        hub = k * (n // len(spokes)) + 7
        to = to[to != hub]
        w = np.full(len(to), 0.25)
        e = sp.coo_matrix((w, (np.full(len(to), hub), to)), shape=(n, n)).tocsr()
        e = e + e.T
        a = a - e + sp.diags(np.asarray(e.sum(axis=1)).ravel())
    a = a.tocsr()
    a.sort_indices()
    return a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data


# level 1: 63,883 rows, of which twelve have 109 to 4,777 entries (a hub row has more than
# 64, its chunks 1,024)
SPOKES = (2500, 700, 160, 90, 60, 50, 40, 40, 30, 30, 25, 20)


@pytest.fixture(scope="module")
def problem():
    rp, ci, va = hubs_in_a_grid(58, SPOKES)
    return rp, ci, va, oracle.Hierarchy(rp, ci, va)


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("batch_cols", [2, 4, 8])
@pytest.mark.parametrize("columns,opt", [(2, {}), (5, {}), (8, {}), (8, {"kcycle_inner": 1}),
                                         (8, {"kcycle_threshold": 0.3})])
def test_batched_hub_rows_bits(amg, problem, precision, batch_cols, columns, opt):
    rp, ci, va, ref = problem
    n = len(rp) - 1
    with amg.Hierarchy(dev(rp), dev(ci), dev(va), max_rhs=8, precision=precision, autotune=0,
                       batch_cols=batch_cols, **opt) as h:
        level = h.export_level(1)
        rows = np.diff(level.row_ptr)
        # two columns are 100,000 values (on level 2 eight are)
        assert 50000 <= level.n < 100000 and 100000 <= 8 * h.level_sizes(2)[0]
        assert rows.max() > 2 * 1024 and ((rows > 256) & (rows < 1024)).any()
        r = dev(np.stack([inputs.rhs(n, 30 + c) for c in range(columns)]))
        z, one = torch.empty_like(r), torch.empty(n, dtype=torch.float64, device="cuda")
        h.kcycle_batch(r, z)
        for c in range(columns):
            h.kcycle(r[c], one)
            assert torch.equal(one, z[c]), c
        if precision == 0 and not opt:
            want = ref.kcycle(inputs.rhs(n, 30))
            np.testing.assert_allclose(z[0].cpu().numpy(), want, rtol=0, atol=1e-10 * np.abs(want).max())
