"""GPU parity of Markov-clustering rows swept in column panels (more products
than a table holds) that the prune empties: the largest entry is kept, whole
rows and single ones, in both step orders and with odd exponents, against the
FP64 oracle step by step."""
import numpy as np
import pytest

from mcl_check import check_mcl_step
from paper_2603_21444_amd import synth
from test_mcl_few import _run

pytestmark = pytest.mark.gpu


def _heavy(n, d, seed, strong):
    """Rows of d random columns; those of the rows in `strong` put most of
    their weight on one."""
    rng = synth.rng_for(seed, 4)
    rows = [np.sort(rng.choice(n, size=d, replace=False)) for _ in range(n)]
    w = [0.5 + rng.random(d) for _ in range(n)]
    for i in strong:
        w[i][int(rng.integers(d))] += 40.0 * d
    ip = np.arange(n + 1, dtype=np.int64) * d
    return synth.HostCSR((n, n), ip, np.concatenate(rows).astype(np.int32),
                         np.concatenate([x / x.sum() for x in w]).astype(np.float32))


@pytest.mark.parametrize("order,r,prune", [("paper", 2, 2e-3), ("paper", 3, 2e-3),
                                           ("workload", 2, 2e-3), ("workload", 3, 2e-3),
                                           ("workload", 1, 2e-3), ("paper", 2, 0.5)])
@pytest.mark.parametrize("strong", [0, 40])
def test_rows_emptied_by_the_prune(order, r, prune, strong):
    X = _heavy(4000, 180, 11, range(0, 4000, 4000 // strong) if strong else ())
    got = _run(X, r=r, prune=prune, topk=100, order=order)
    check_mcl_step(X, got, r, prune, 100, order=order, rows=np.arange(0, 4000, 20))
    if not strong and (order == "paper" or r < 3):  # (the cube lifts entries over the prune)
        assert (np.diff(got.indptr) == 1).mean() > 0.9
