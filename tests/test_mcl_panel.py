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


def _few_per_panel(n, entries, length, seed, zero=()):
    """60 rows of `entries` entries, each a row of `length` random columns of
    n; the rows in `zero` point to rows of zeros; all other rows are empty."""
    rng = synth.rng_for(seed, 4)
    hubs = 2 * entries
    rows = [np.zeros(0, dtype=np.int64)] * n
    vals = [np.zeros(0)] * n
    at = rng.permutation(n)[:hubs + 60]
    hub, zeros = at[:hubs - entries // 2], at[hubs - entries // 2:hubs]
    for v in at[:hubs]:
        rows[v] = np.sort(rng.choice(n, size=length, replace=False))
        vals[v] = (0.5 + rng.random(length)) * (0.0 if v in set(zeros.tolist()) else 1.0)
    body = at[hubs:]
    for t, v in enumerate(body):
        pick = np.concatenate([zeros, zeros]) if t in zero else hub
        pick = np.unique(pick)
        rows[v] = np.sort(rng.choice(pick, size=min(entries, pick.size), replace=False))
        vals[v] = 0.5 + rng.random(rows[v].size)
    ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    v = np.concatenate([x / max(x.sum(), 1e-30) for x in vals])
    return synth.HostCSR((n, n), ip, np.concatenate(rows).astype(np.int32), v.astype(np.float32)), body


@pytest.mark.parametrize("entries,length", [(200, 100), (40, 600), (1500, 12)])
@pytest.mark.parametrize("order,r,prune,topk", [("workload", 2, 1e-5, 10000), ("workload", 3, 1e-9, 500),
                                                ("workload", 2, 0.0, 300), ("paper", 2, 4e-5, 300),
                                                ("paper", 2, 0.5, 100)])
def test_few_products_per_panel(entries, length, order, r, prune, topk):
    """Some 20000 products on 300000 columns (19 panels): only the marked
    columns are looked at; entries in LDS and in the slot scratch, all order
    and prune combinations, rows that the prune empties."""
    X, body = _few_per_panel(300000, entries, length, entries)
    got = _run(X, r=r, prune=prune, topk=topk, order=order)
    lens = np.diff(got.indptr)
    assert lens[body].all()
    if prune == 0.5:
        assert (lens[body] == 1).all()
    check_mcl_step(X, got, r, prune, topk, order=order, rows=np.sort(body))
