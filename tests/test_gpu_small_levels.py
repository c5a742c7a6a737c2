"""The small levels of a hierarchy on the GPU against the oracle: levels that one
workgroup holds (any depth, row length and coarsest solve), star levels above a
single coarse unknown, the one-launch aggregation and the scans at the sizes where
their paths change.

Hierarchies must be the oracle's bit for bit; one K-cycle agrees with it to 1e-10 of
its largest entry (the tolerance of the other K-cycle tests: only the order of the
sums differs).
"""
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


def laplacian(n, i, j, w, shift):
    """CSR of the weighted graph Laplacian of the edges (i, j) plus shift on the diagonal."""
    a = sp.coo_matrix((np.concatenate([-w, -w]), (np.concatenate([i, j]), np.concatenate([j, i]))), shape=(n, n))
    a = a.tocsr()
    a = (a + sp.diags(shift - np.asarray(a.sum(axis=1)).ravel())).tocsr()
    a.sort_indices()
    return a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data.astype(np.float64)


def star_graph(arms, chains=0, seed=4):
    """A hub joined to `arms` vertices, each joined to one more: the hub aggregates its
    neighbours, so level 1 is a star of arms + 1 rows (and level 2 one unknown).  Each
    chain joins the ends of two arms through two more vertices, which become edges
    between leaves of the star."""
    n = 1 + 2 * arms + 2 * chains
    near, end = np.arange(1, arms + 1), np.arange(arms + 1, 2 * arms + 1)
    i, j = [np.zeros(arms, np.int64), near], [near, end]
    for c in range(chains):
        a, b = 2 * arms + 1 + 2 * c, 2 * arms + 2 + 2 * c
        i.append(np.array([end[2 * c], a, b]))
        j.append(np.array([a, b, end[2 * c + 1]]))
    i, j = np.concatenate(i), np.concatenate(j)
    w = 0.5 + inputs.uniform(seed, np.arange(len(i), dtype=np.uint64))
    return laplacian(n, i, j, w, 1e-2)


def hub_and_grid(side, spokes):
    """A 2D grid whose first vertex is also joined to `spokes` others."""
    rp, ci, va = inputs.grid_laplacian((side, side), jitter=0.2, seed=6)
    n = len(rp) - 1
    t = np.arange(n // 2, n // 2 + spokes)
    w = np.full(spokes, 0.25)
    b = sp.csr_matrix((va, ci, rp), shape=(n, n))
    r, c, v = laplacian(n, np.zeros(spokes, np.int64), t, w, 0.0)
    a = (b + sp.csr_matrix((v, c, r), shape=(n, n))).tocsr()
    a.sort_indices()
    return a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data


def check(amg, csr, columns=1, **opt):
    rp, ci, va = csr
    n = len(rp) - 1
    h = amg.Hierarchy(dev(rp), dev(ci), dev(va), max_rhs=columns, **opt)
    ref = oracle.Hierarchy(rp, ci, va, **{k: v for k, v in opt.items() if k not in ("precision", "use_graph")})
    print(f"[small] levels {[h.level_sizes(l)[:2] for l in range(h.num_levels)]} opt {opt}", flush=True)
    assert h.num_levels == ref.num_levels
    for l in range(h.num_levels):
        g, o = h.export_level(l), ref.level(l)
        assert (g.n, g.nnz, g.passes) == (o.n, o.nnz, o.passes), l
        for what in ("agg", "row_ptr", "col", "val"):
            np.testing.assert_array_equal(getattr(g, what), getattr(o, what), err_msg=f"level {l} {what}")
    r = np.stack([inputs.rhs(n, 3 + c) for c in range(columns)])
    z = torch.empty((columns, n), dtype=torch.float64, device="cuda")
    h.kcycle_batch(dev(r), z)
    for c in range(columns):
        zo = ref.kcycle(r[c])
        np.testing.assert_allclose(z[c].cpu().numpy(), zo, rtol=0, atol=1e-10 * np.abs(zo).max())
        one = torch.empty(n, dtype=torch.float64, device="cuda")
        h.kcycle(dev(r[c]), one)
        assert torch.equal(one, z[c])  # a column of a batch has the bits it has alone
    return h, ref


HELD = {
    # two levels above the coarsest on two and four slots per thread, six on one (9x9: none)
    "grid_9x9": (lambda: inputs.grid_laplacian((9, 9), jitter=0.2, seed=1), {}),
    "grid_25x24": (lambda: inputs.grid_laplacian((25, 24), jitter=0.2, seed=1), {}),
    "grid_45x45": (lambda: inputs.grid_laplacian((45, 45), jitter=0.2, seed=1), {}),
    "grid_131x67": (lambda: inputs.grid_laplacian((131, 67), jitter=0.2, seed=1), {}),
    "path_8000": (lambda: inputs.grid_laplacian((8000,), jitter=0.2, seed=1), {"coarsest_size": 2}),
    # more small levels than one workgroup takes
    "path_2000_pairs": (lambda: inputs.grid_laplacian((2000,), jitter=0.2, seed=1),
                        {"coarsest_size": 2, "max_aggregate": 2}),
    # rows of 1, 2, 4, 16 and 64 lanes (dense_200: two levels, nothing held)
    "dense_200": (lambda: inputs.random_graph_laplacian(200, 0.4, 5, False), {"coarsest_size": 8}),
    "hub_40": (lambda: hub_and_grid(40, 40), {}),
    "hub_257": (lambda: hub_and_grid(40, 257), {}),
    "hub_700": (lambda: hub_and_grid(40, 700), {"max_aggregate": 3}),
    # isolated vertices (graph_sparse: more than a workgroup takes), and a star on its own
    "graph_3000": (lambda: inputs.rgg_laplacian(3000, seed=5, weight_range=(0.5, 1.5)), {}),
    "graph_sparse": (lambda: inputs.rgg_laplacian(4000, mean_degree=3.0, seed=5), {}),
    "star_600": (lambda: star_graph(600, 5), {"coarsest_size": 1}),
}


@pytest.mark.parametrize("opt", [{}, {"kcycle_inner": 1}, {"kcycle_threshold": 0.3}], ids=["nu2", "nu1", "theta"])
@pytest.mark.parametrize("name", sorted(HELD))
def test_levels_held_by_one_workgroup(amg, name, opt):
    make, base = HELD[name]
    h, _ = check(amg, make(), columns=3 if not opt else 1, **base, **opt)
    h.close()


# one row either side of the counts of rows per thread, of the largest star that a block
# takes, and edges between leaves
@pytest.mark.parametrize("arms,chains", [(2046, 0), (2047, 0), (2048, 0), (2060, 9), (5119, 0), (5120, 3), (6000, 12),
                                         (8191, 0), (8192, 0), (3000, 60)])
def test_star_level(amg, arms, chains):
    opts = [{}] if arms != 2060 else [{}, {"kcycle_inner": 1}, {"kcycle_threshold": 0.3}]
    for opt in opts:
        h, ref = check(amg, star_graph(arms, chains), columns=2, coarsest_size=1, max_levels=3, **opt)
        n = h.n
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        b = inputs.rhs(n, 8)
        st, info = h.solve(dev(b), x, tol=1e-9)
        assert st == amg.AMG_OK and info.rel_residual <= 1e-9
        h.close()


# around the capacity of the one-launch aggregation, of the one-block scan and of the
# one-block search for long rows
@pytest.mark.parametrize("n,cap", [(65, 0), (1024, 2), (6200, 0), (6290, 3), (6400, 0), (16384, 0), (16385, 0)])
def test_small_setup_edges(amg, n, cap):
    h, _ = check(amg, inputs.grid_laplacian((n,), jitter=0.3, seed=n), max_aggregate=cap, kcycle_inner=1)
    h.close()


# the coarsest inverse: sizes around its lanes and its capacity, a single level
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65])
def test_coarsest_inverse(amg, n):
    rp, ci, va = inputs.random_graph_laplacian(n, 0.3, 11 + n, False)
    h = amg.Hierarchy(dev(rp), dev(ci), dev(va), max_levels=1)
    b = inputs.rhs(n, 5)
    z = torch.empty(n, dtype=torch.float64, device="cuda")
    h.kcycle(dev(b), z)
    x = np.linalg.solve(inputs.csr_to_dense(rp, ci, va), b)
    np.testing.assert_allclose(z.cpu().numpy(), x, rtol=0, atol=1e-12 * np.abs(x).max())
    h.close()


# mid-size levels of a batch are smoothed in two launches (here level 1 from three columns
# on), those of a single column in one
@pytest.mark.parametrize("columns", [2, 5, 8])
@pytest.mark.parametrize("precision", [0, 1])
def test_batched_mid_level_bits(amg, columns, precision):
    rp, ci, va = inputs.grid_laplacian((50, 49, 48), jitter=0.1, seed=9)
    n = len(rp) - 1
    h = amg.Hierarchy(dev(rp), dev(ci), dev(va), max_rhs=8, precision=precision, autotune=0)
    r = dev(np.stack([inputs.rhs(n, 30 + c) for c in range(columns)]))
    z = torch.empty_like(r)
    h.kcycle_batch(r, z)
    one = torch.empty(n, dtype=torch.float64, device="cuda")
    for c in range(columns):
        h.kcycle(r[c], one)
        assert torch.equal(one, z[c]), c
    h.close()


# A cycle of three launches runs on the caller's vectors unless they overlap: apart,
# at odd offsets, the same and shifted against each other the result has the same bits.
@pytest.mark.parametrize("problem", ["held", "star"])
def test_short_cycle_on_the_callers_vectors(amg, problem):
    csr = inputs.grid_laplacian((33, 31), jitter=0.1, seed=3) if problem == "held" else star_graph(300)
    n = len(csr[0]) - 1
    b = np.random.default_rng(7).standard_normal(n)
    with amg.Hierarchy(*(torch.from_numpy(v).cuda() for v in csr)) as h:
        want = torch.empty(n, dtype=torch.float64, device="cuda")
        h.kcycle(torch.from_numpy(b).cuda(), want)
        for at_r, at_z in [(0, n), (1, n + 3), (n + 5, 1), (0, 0), (1, 0), (0, 1), (0, n - 1), (n - 1, 0)]:
            room = torch.full((2 * n + 8,), 7.0, dtype=torch.float64, device="cuda")
            r, z = room[at_r : at_r + n], room[at_z : at_z + n]
            r.copy_(torch.from_numpy(b))
            h.kcycle(r, z)
            assert torch.equal(z, want), (at_r, at_z)
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        h.solve(want, x, 1e-8)
        h.kcycle(torch.from_numpy(b).cuda(), x)  # after a solve, whose graph holds the cycle too
        assert torch.equal(x, want)
