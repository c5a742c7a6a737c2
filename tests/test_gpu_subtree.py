"""The last levels of a hierarchy in one workgroup, in every form that they take (depth,
slots per thread, lanes per row, long rows, decoupled unknowns, FP32 storage), star
levels in FP32 storage, and residuals so small that a level's products are subnormal
numbers.  The form that a case takes is computed from its levels and asserted.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sp = pytest.importorskip("scipy.sparse")
pytest.importorskip("scipy.sparse.linalg")

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


def held(level, last, value_bytes=8):
    """What the library's rules make of a hierarchy's last levels, from the exported
    levels alone: None when no level is held by one workgroup, else its depth (levels
    above the coarsest), the slots per thread on the top one, the classes of lanes per row
    (c: 2^c lanes, 7: more entries than a wavefront takes), the rows of class 7 and the
    coupled and decoupled unknowns of the coarsest level."""
    threads, unroll, lds = 512, 4, 160 * 1024 - 512
    coarsest = level(last)
    lengths = np.diff(coarsest.row_ptr)
    alone = (lengths == 1) & (np.bincount(coarsest.col, minlength=coarsest.n) == 1) & (coarsest.n > 64)
    decoupled = int(alone.sum())
    if coarsest.n - decoupled > 64 or decoupled > threads:
        return None
    levels = []  # the coarsest's upper neighbours, coarsest first
    while len(levels) < 6 and last - 1 - len(levels) >= 1 and level(last - 1 - len(levels)).n <= 4096:
        levels.append(level(last - 1 - len(levels)))
    waves, long_rows, extra, classes = [], [], [], []
    for k, e in enumerate(levels):
        rows = np.diff(e.row_ptr)
        members = np.bincount(levels[k + 1].agg, minlength=e.n) if k + 1 < len(levels) else np.ones(e.n, int)
        lanes = np.maximum(-(-rows // unroll), -(-members // (2 * unroll)))
        c = np.where(rows > 64 * unroll, 7, np.clip(np.ceil(np.log2(np.maximum(lanes, 1))), 0, 6).astype(int))
        waves.append(-(-int((1 << np.minimum(c, 6)).sum()) // 64))
        long_rows.append(int((c == 7).sum()))
        extra.append(int((rows[c == 7] - 64 * unroll).sum()))
        classes.append(set(c.tolist()))
    depth = 0
    for k in range(len(levels)):
        if waves[k] <= 32:
            depth = k + 1
        if waves[k] > 8:
            break
    for depth in range(depth, 0, -1):
        width = 1 if waves[depth - 1] <= 8 else 2 if waves[depth - 1] <= 16 else 4
        vector = lambda slots: 8 * (slots * threads + 1)
        used = 8 * 64 + 8 * (64 + threads) + (depth - 1) * 3 * vector(1) + 4 * vector(width)
        used += sum(4 * (long_rows[k] + 1) + (value_bytes + 2) * extra[k] + 21 for k in range(depth))
        if used <= lds:
            return {"depth": depth, "width": width, "classes": set().union(*classes[:depth]),
                    "long": sum(long_rows[:depth]), "coupled": coarsest.n - decoupled, "decoupled": decoupled}
    return None


def spiders(hubs, arms, length, chains=0):
    """`hubs` vertices in a row, two others between neighbours, each with `arms` paths of
    `length` vertices: a hub takes its neighbours on every level, so its row stays long.
    Each of the `chains` joins the ends of two paths through two more vertices."""
    i, j, n = [], [], hubs
    for h in range(hubs):
        v = n + np.arange(arms * length).reshape(arms, length)
        i += [np.full(arms, h), v[:, :-1].ravel()]
        j += [v[:, 0], v[:, 1:].ravel()]
        n += arms * length
        if h + 1 < hubs:
            i.append(np.array([h, n, n + 1]))
            j.append(np.array([n, n + 1, h + 1]))
            n += 2
    for c in range(chains):
        i.append(np.array([v[2 * c, -1], n, n + 1]))
        j.append(np.array([n, n + 1, v[2 * c + 1, -1]]))
        n += 2
    i, j = np.concatenate(i), np.concatenate(j)
    w = 0.5 + inputs.uniform(4, np.arange(len(i), dtype=np.uint64))
    a = sp.coo_matrix((np.concatenate([-w, -w]), (np.concatenate([i, j]), np.concatenate([j, i]))), shape=(n, n))
    a = a.tocsr()
    a = (a + sp.diags(0.5 - np.asarray(a.sum(axis=1)).ravel())).tocsr()
    a.sort_indices()
    return a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data


def paths(count, length):
    """Separate paths: each ends as one decoupled unknown."""
    rp, ci, va = inputs.grid_laplacian((length,), jitter=0.2, seed=2)
    a = sp.block_diag([sp.csr_matrix((va * (1 + 0.01 * k), ci, rp)) for k in range(count)], format="csr")
    a.sort_indices()
    return a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data


def grid(*dims):
    return lambda: inputs.grid_laplacian(dims, jitter=0.2, seed=1)


def graph(n, degree):
    def make():
        rp, ci, va = inputs.rgg_laplacian(n, mean_degree=degree, seed=5)
        return rp, ci, va + 0.5 * (ci == np.repeat(np.arange(n), np.diff(rp)))
    return make


# problem, options, and what of held() the case is there for
PATHS = {
    # depth and slots per thread
    "1x1": (grid(16, 16), {}, {"depth": 1, "width": 1}),
    "2x1": (grid(20, 20), {"max_aggregate": 3}, {"depth": 2, "width": 1}),
    "3x1": (grid(10, 10), {"coarsest_size": 1}, {"depth": 3, "width": 1}),
    "4x1": (grid(20, 20), {"coarsest_size": 1}, {"depth": 4, "width": 1}),
    "5x1": (grid(10, 10), {"coarsest_size": 1, "max_aggregate": 3}, {"depth": 5, "width": 1}),
    "6x1": (grid(300), {"coarsest_size": 2}, {"depth": 6, "width": 1}),
    "1x2": (grid(16, 16, 16), {"max_aggregate": 3}, {"depth": 1, "width": 2}),
    "2x2": (grid(33, 31), {}, {"depth": 2, "width": 2}),
    "3x2": (grid(33, 31), {"max_aggregate": 3}, {"depth": 3, "width": 2}),
    "4x2": (grid(25, 24), {"coarsest_size": 8}, {"depth": 4, "width": 2}),
    "5x2": (grid(25, 24), {"coarsest_size": 1}, {"depth": 5, "width": 2}),
    "6x2": (grid(270, 3), {"coarsest_size": 1}, {"depth": 6, "width": 2}),
    "1x4": (lambda: spiders(1, 1500, 2, 60), {"coarsest_size": 1}, {"depth": 1, "width": 4, "long": 1}),
    "2x4": (grid(45, 45), {}, {"depth": 2, "width": 4}),
    "3x4": (grid(90, 90), {"coarsest_size": 8}, {"depth": 3, "width": 4}),
    "4x4": (grid(45, 45), {"coarsest_size": 8}, {"depth": 4, "width": 4}),
    "5x4": (grid(45, 45), {"coarsest_size": 1}, {"depth": 5, "width": 4}),
    "6x4": (grid(37, 37), {"coarsest_size": 1, "max_aggregate": 4}, {"depth": 6, "width": 4}),
    # lanes per row: 32 and 64 of them, and rows that are longer still, on one and two levels
    "32 lanes": (grid(24, 24, 24), {}, {"classes": {0, 1, 2, 3, 4, 5}}),
    "long rows, 2 slots": (lambda: spiders(1, 350, 6), {"coarsest_size": 1}, {"width": 2, "long": 2}),
    "long rows, 4 slots": (lambda: spiders(1, 300, 10), {"coarsest_size": 1}, {"width": 4, "long": 2}),
    "three long rows": (lambda: spiders(2, 300, 3), {"coarsest_size": 1}, {"width": 2, "long": 3}),
    "64 lanes": (lambda: spiders(1, 400, 20), {"coarsest_size": 1}, {"depth": 3, "long": 2, "classes": {0, 6, 7}}),
    # decoupled coarsest unknowns with 1, 2, 4 and 8 lanes, and nothing but them
    "393 decoupled": (graph(2500, 3.0), {}, {"coupled": 25, "decoupled": 393}),
    "175 decoupled": (graph(3000, 4.0), {}, {"coupled": 19, "decoupled": 175}),
    "70 decoupled": (graph(1000, 4.0), {}, {"coupled": 9, "decoupled": 70}),
    "62 decoupled": (graph(3000, 5.0), {}, {"coupled": 6, "decoupled": 62}),
    "all decoupled": (lambda: paths(120, 8), {}, {"coupled": 0, "decoupled": 120}),
}


def fp32_tolerance(rp, ci, va):
    """Rounding the entries of A to FP32 moves the solution of a system by at most 2^-24
    times the largest entry of |A^-1| |A| 1, relative to its own largest entry (|A^-1| is
    A^-1 for an M-matrix).  32 of them for the coarse matrices and the vectors that are
    rounded too."""
    a = sp.csr_matrix((va, ci, rp))
    return 32 * 2.0**-24 * sp.linalg.spsolve(a.tocsc(), np.asarray(abs(a).sum(axis=1)).ravel()).max()


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(PATHS))
def test_every_form(amg, name, precision):
    make, opt, want = PATHS[name]
    rp, ci, va = make()
    n = len(rp) - 1
    ref = oracle.Hierarchy(rp, ci, va, **opt)
    with amg.Hierarchy(dev(rp), dev(ci), dev(va), precision=precision, max_rhs=2, **opt) as h:
        got = held(h.export_level, h.num_levels - 1, 4 if precision else 8)
        print(f"[subtree] {name} {got}", flush=True)
        assert got is not None and {k: got[k] for k in want} == want
        tol = fp32_tolerance(rp, ci, va) if precision else 1e-10
        r = np.stack([inputs.rhs(n, 3), inputs.rhs(n, 4)])
        z, one = torch.empty((2, n), dtype=torch.float64, device="cuda"), torch.empty(n, dtype=torch.float64, device="cuda")
        h.kcycle_batch(dev(r), z)
        for c in range(2):
            zo = ref.kcycle(r[c])
            np.testing.assert_allclose(z[c].cpu().numpy(), zo, rtol=0, atol=tol * np.abs(zo).max())
            h.kcycle(dev(r[c]), one)
            assert torch.equal(one, z[c])


# star levels in FP32: two, five and eight rows per thread, with and without edges
# between the leaves
@pytest.mark.parametrize("arms,chains", [(1500, 0), (1500, 9), (4000, 0), (4000, 9), (8000, 0), (8000, 9)])
def test_star_level_in_fp32(amg, arms, chains):
    rp, ci, va = spiders(1, arms, 2, chains)
    n = len(rp) - 1
    zo = oracle.Hierarchy(rp, ci, va, coarsest_size=1, max_levels=3).kcycle(inputs.rhs(n, 3))
    with amg.Hierarchy(dev(rp), dev(ci), dev(va), precision=1, coarsest_size=1, max_levels=3) as h:
        assert [h.level_sizes(l)[0] for l in (1, 2)] == [arms + 1, 1]
        z = torch.empty(n, dtype=torch.float64, device="cuda")
        h.kcycle(dev(inputs.rhs(n, 3)), z)
    np.testing.assert_allclose(z.cpu().numpy(), zo, rtol=0, atol=fp32_tolerance(rp, ci, va) * np.abs(zo).max())


# The K-cycle is homogeneous: of 2^-514 r it is 2^-514 times that of r.  The products
# (c, A c) are then 2^-1028 times theirs, subnormal numbers whose reciprocals overflow.
# Tolerance: a sum of at most 2^10 such products is off by at most 2^10 2^-1075, which is
# 2^-27 of a product of 2^-10 (the smallest expected, for a residual of entries up to 1);
# two orders for the quotients and levels that it passes through.
@pytest.mark.parametrize("dims,opt", [((33, 31), {}), ((45, 45), {}), ((12, 12, 12), {}),
                                      ((60, 60), {"coarsest_size": 1})])
def test_kcycle_of_a_tiny_residual(amg, dims, opt):
    rp, ci, va = inputs.grid_laplacian(dims, jitter=0.1, seed=3)
    n = len(rp) - 1
    r = inputs.rhs(n, 7)
    want = oracle.Hierarchy(rp, ci, va, **opt).kcycle(r)
    z = torch.empty(n, dtype=torch.float64, device="cuda")
    with amg.Hierarchy(dev(rp), dev(ci), dev(va), **opt) as h:
        h.kcycle(dev(np.ldexp(r, -514)), z)
    np.testing.assert_allclose(np.ldexp(z.cpu().numpy(), 514), want, rtol=0, atol=1e-6 * np.abs(want).max())
