"""GPU numeric pass on a B whose columns changed after the symbolic pass: a row
without repeated columns gains one, so that it has as many products as before
and one distinct column less.  Every kernel that can take the row flags it."""
import numpy as np
import pytest

from paper_2603_21444_amd import synth

pytestmark = pytest.mark.gpu


def _disjoint(products, n, clustered, seed):
    """A: one row of some entries (and a few short rows); B rows of uneven
    lengths whose columns, over all of them, differ: `products` of n."""
    rng = synth.rng_for(seed, 9)
    if clustered:
        cols = rng.integers(n - products) + rng.permutation(products)
    else:
        cols = rng.choice(n, size=products, replace=False)
    cuts = np.sort(rng.choice(np.arange(1, products), size=max(1, products // 7), replace=False))
    rows = [np.sort(r) for r in np.split(cols.astype(np.int32), cuts)]
    k = len(rows)
    B = synth.HostCSR((k, n), np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64),
                      np.concatenate(rows), rng.standard_normal(products))
    A = synth.HostCSR((5, k), np.array([0, 1, 1, 1 + k, 2 + k, 2 + k]),
                      np.concatenate([[0], np.arange(k), [k - 1]]).astype(np.int32),
                      rng.standard_normal(k + 2))
    return A, B


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("products,n", [(14, 5000), (30, 5000), (60, 5000), (125, 1 << 20),
                                        (250, 1 << 20), (500, 1 << 20), (1000, 1 << 20),
                                        (2000, 1 << 20), (4000, 1 << 20), (8000, 1 << 20),
                                        (12000, 1 << 20), (12000, 1 << 14), (9000, 1 << 23),
                                        (250, 1 << 25), (2000, 1 << 25)])
@pytest.mark.parametrize("clustered", [False, True])
def test_a_repeat_is_flagged(products, n, clustered, dtype):
    import torch
    from paper_2603_21444_amd import binding
    hA, hB = _disjoint(products, n, clustered, products)
    A, B = binding.to_device(hA.astype(dtype)), binding.to_device(hB.astype(dtype))
    plan = binding.Plan()
    rp, nnz = plan.symbolic([A], [B])
    assert nnz == products + (hB.indptr[1] - hB.indptr[0]) + (hB.indptr[-1] - hB.indptr[-2])
    plan.numeric([A], [B], rp, nnz)
    assert plan.status() == binding.SPG_OK
    # the column of another row of B nearest to the first row's first one becomes that
    first = int(hB.indptr[1])
    at = first + int(np.abs(hB.indices[first:] - hB.indices[0]).argmin())
    B.col_idx[at] = int(hB.indices[0])
    plan.numeric([A], [B], rp, nnz)
    torch.cuda.synchronize()
    assert plan.status() == binding.SPG_ERR_INVALID
