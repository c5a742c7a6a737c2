"""Aggregation of an asymmetric pattern whose overlapping claims add up to the number of
rows while one row is left over: an error, not an aggregate read from nowhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def amg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1302_2547_amd import amg as mod
    return mod


def overlapping(triples):
    """Rows {0, 2, 3}, {0, 1}, {1, 2}, {3}: the first pass takes rows 0 and 3, which both
    claim row 3 -- four claims, none of row 1 (the degrees alone decide) -- and every
    triple's middle row, which claims its two neighbours."""
    rows = [[0, 2, 3], [0, 1], [1, 2], [3]]
    for k in range(4, 4 + 3 * triples, 3):
        rows += [[k, k + 1], [k, k + 1, k + 2], [k + 1, k + 2]]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    va = np.where(ci == np.repeat(np.arange(len(rows)), np.diff(rp)), 4.0, -1.0)
    return rp, ci, va


# aggregated in one launch, and by separate passes
@pytest.mark.parametrize("triples", [30, 30000])
def test_overlapping_claims_are_an_error(amg, triples):
    csr = [torch.from_numpy(v).cuda() for v in overlapping(triples)]
    with pytest.raises(amg.AmgError) as e:
        amg.Hierarchy(*csr, coarsest_size=1)
    assert e.value.status == amg.AMG_ERR_DEVICE
