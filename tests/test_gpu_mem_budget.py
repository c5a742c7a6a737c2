"""Memory budgets: a hierarchy gives up its optional structures (one-workgroup levels,
star layouts, iterates of the batched post-smoothing) before setup is refused.

LEAST holds, per problem, a budget of the matrices, the layouts that every solve
reads and the work vectors, without any optional structure; every budget from it on is
enough, and amg_memory_bytes never exceeds it.
"""
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def grid(*dims):
    return lambda: inputs.grid_laplacian(dims, jitter=0.1, seed=3)


LEAST = {
    "45x45": (grid(45, 45), {}, 9331084),
    "181x173": (grid(181, 173), {}, 27245828),
    "41x37x29": (grid(41, 37, 29), {}, 40259712),
    "64x64 to one unknown": (grid(64, 64), {"coarsest_size": 1}, 17848252),
    "graph 20000": (lambda: inputs.rgg_laplacian(20000, seed=5, weight_range=(0.5, 1.5)), {}, 22190772),
    "sparse graph 3000": (lambda: inputs.rgg_laplacian(3000, mean_degree=4.0, seed=5), {}, 11202540),
}


def budgets(amg, make, opt, least):
    """Sets up and solves with `least` bytes and with more, up to where all optional
    structures fit."""
    rp, ci, va = make()
    n, columns = len(rp) - 1, opt.get("max_rhs", 1)
    csr = dev(rp), dev(ci), dev(va)
    b = dev(np.stack([inputs.rhs(n, 20 + c) for c in range(columns)]))
    with amg.Hierarchy(*csr, autotune=0, **opt) as h:
        most = max(h.memory_bytes + least // 8, least)
    x = torch.empty_like(b)
    for budget in np.linspace(least, most, 25).astype(np.int64):
        print(f"[budget] {budget}", flush=True)
        with amg.Hierarchy(*csr, mem_budget=int(budget), autotune=0, **opt) as h:
            assert h.memory_bytes <= budget
            x.zero_()
            st, infos = h.solve_batch(b, x, 1e-8)
            assert st == amg.AMG_OK and max(i.rel_residual for i in infos) <= 1e-8


@pytest.mark.parametrize("name", sorted(LEAST))
def test_budget_without_optional_structures(amg, name):
    budgets(amg, *LEAST[name])


# the same for several right-hand sides, where the mid-size levels' iterates are optional
LEAST_BATCH = {
    "60^3 x 8": (grid(60, 60, 60), {"max_rhs": 8}, 367024888),
    "60^3 x 8 mixed": (grid(60, 60, 60), {"max_rhs": 8, "precision": 1}, 419577356),
    "200x200 x 4": (grid(200, 200), {"max_rhs": 4}, 85811564),
    "graph 20000 x 8": (lambda: inputs.rgg_laplacian(20000, seed=5, weight_range=(0.5, 1.5)), {"max_rhs": 8},
                        112240144),
}


@pytest.mark.parametrize("name", sorted(LEAST_BATCH))
def test_budget_of_a_batch(amg, name):
    budgets(amg, *LEAST_BATCH[name])


def test_no_iterates_for_one_column_per_block(amg):
    """The iterates of 41,000 rows x 8 columns are held only where a batched sweep reads
    them: not with one column per block."""
    csr = [dev(v) for v in inputs.grid_laplacian((50, 49, 48), jitter=0.1, seed=9)]
    held = []
    for cb in (1, 4):
        with amg.Hierarchy(*csr, max_rhs=8, batch_cols=cb, autotune=0) as h:
            rows = [h.level_sizes(l)[0] for l in range(h.num_levels)]
            held.append(h.memory_bytes)
    mid = [n for n in rows[1:] if n < 100000 and 8 * n >= 100000]
    assert mid and held[1] - held[0] == 8 * 8 * sum(mid)
