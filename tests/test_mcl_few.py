"""GPU parity of Markov-clustering rows that fall on few columns: clusters of
various sizes under random labels (up to and past the 512 columns that one
block holds), rows with thousands of columns between them, top-k cuts, ties,
no prune, both step orders, against the FP64 oracle step by step."""
import numpy as np
import pytest

from mcl_check import check_mcl_step
from paper_2603_21444_amd import synth

pytestmark = pytest.mark.gpu


def _clusters(sizes, seed, weights="u", spread=0):
    """Row-stochastic X whose clusters hold sizes[c] vertices each (labels
    shuffled); the first `spread` rows hold 60 random columns instead."""
    n = int(sum(sizes))
    rng = synth.rng_for(seed, 2)
    label = rng.permutation(n)
    rows = [None] * n
    base = 0
    for c in sizes:
        members = np.sort(label[base:base + c])
        for v in label[base:base + c]:
            rows[v] = members
        base += c
    for v in range(spread):
        rows[v] = np.sort(rng.choice(n, size=60, replace=False))
    w = [np.ones(r.size) if weights == "equal" else 0.5 + 0.5 * rng.random(r.size) for r in rows]
    ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    return synth.HostCSR((n, n), ip, np.concatenate(rows).astype(np.int32),
                         np.concatenate([x / x.sum() for x in w]).astype(np.float32))


def _run(X, **kw):
    import torch
    from paper_2603_21444_amd import binding
    plan = binding.Plan()
    got = binding.mcl_iteration(binding.to_device(X), plan=plan, **kw)
    torch.cuda.synchronize()
    assert plan.status() == binding.SPG_OK
    return got.to_host()


@pytest.mark.parametrize("order,prune,topk", [("workload", 1e-4, 1000), ("workload", 0.0, 30),
                                              ("paper", 1e-3, 500), ("paper", 0.0, 7)])
def test_clusters_of_many_sizes(order, prune, topk):
    sizes = [17, 20, 33, 64, 90, 128, 200] * 6 + [40] * 30
    X = _clusters(sizes, 3)
    check_mcl_step(X, _run(X, r=2, prune=prune, topk=topk, order=order), 2, prune, topk, order=order)


def test_rows_at_the_limit_of_columns():
    """512 columns are held, 513 are given back; both in one bin with rows
    that are given back for having thousands."""
    X = _clusters([512, 513, 511, 100, 30, 30, 30], 5, spread=150)
    check_mcl_step(X, _run(X, r=2, prune=1e-5, topk=1000), 2, 1e-5, 1000)


@pytest.mark.parametrize("topk", [1, 5, 64])
def test_ties_keep_the_smallest_columns(topk):
    X = _clusters([64, 128, 32] * 4, 7, weights="equal")
    got = _run(X, r=2, prune=1e-4, topk=topk)
    lens = np.diff(X.indptr)
    for i in range(X.shape[0]):
        k = min(topk, int(lens[i]))
        c, v = got.row(i)
        assert np.array_equal(c, X.row(i)[0][:k]), i
        assert np.allclose(v, 1.0 / k, rtol=1e-6)


def test_many_rows_given_back():
    """Most rows have more columns than a block holds: after the first
    hundreds the rest of the bin is left to the hash kernel."""
    X = _clusters([25] * 200, 9, spread=4000)
    check_mcl_step(X, _run(X, r=2, prune=1e-6, topk=4000), 2, 1e-6, 4000, rows=np.arange(0, 5000, 3))


def _scaled_columns(decades, seed):
    """Clusters of 40 and 90 vertices whose columns differ in size by up to
    10^decades, the same in all rows."""
    X = _clusters([40] * 20 + [90] * 8, seed)
    scale = 10.0 ** -(decades * synth.rng_for(seed, 5).random(X.shape[0]))
    v = X.data.astype(np.float64) * scale[X.indices]
    rows = np.repeat(np.arange(X.shape[0]), np.diff(X.indptr))
    v /= np.bincount(rows, weights=v)[rows]
    return X.with_data(v.astype(np.float32))


@pytest.mark.parametrize("decades", [4, 9, 14, 18])
def test_entries_of_very_different_size_without_a_prune(decades):
    """Every entry is kept: entries far below the row's sum are as accurate as
    FP32 sums."""
    X = _scaled_columns(decades, 13)
    check_mcl_step(X, _run(X, r=1, prune=0.0, topk=1000), 1, 0.0, 1000)


def test_rows_of_zeros_and_underflow():
    """Rows whose stored values are zero, and rows whose inflated values
    underflow, have no entries, as in the hash kernel; their neighbours are
    the oracle's."""
    X = _clusters([64] * 12, 17)
    v = X.data.copy()
    zero, tiny = np.arange(0, X.shape[0], 5), np.arange(1, X.shape[0], 5)
    for i in zero:
        v[X.indptr[i]:X.indptr[i + 1]] = 0.0
    for i in tiny:
        v[X.indptr[i]:X.indptr[i + 1]] *= 1e-30
    X = X.with_data(v)
    got = _run(X, r=2, prune=1e-4, topk=1000)
    lens = np.diff(got.indptr)
    assert not lens[zero].any() and not lens[tiny].any()
    check_mcl_step(X, got, 2, 1e-4, 1000, rows=np.arange(2, X.shape[0], 5))


def _rows_of(n, d, seed, clustered):
    """n rows of d entries: clusters of d vertices (labels shuffled) for the
    rows in `clustered`, d random columns for the others."""
    rng = synth.rng_for(seed, 6)
    label = rng.permutation(n)
    at = np.argsort(label)
    cols = np.sort(label[np.minimum(at // d * d, n - d)[:, None] + np.arange(d)], axis=1)
    wide = np.ones(n, dtype=bool)
    wide[clustered] = False
    for i in np.nonzero(wide)[0]:
        cols[i] = np.sort(rng.choice(n, size=d, replace=False))
    w = 0.5 + 0.5 * rng.random((n, d))
    w /= w.sum(1, keepdims=True)
    return synth.HostCSR((n, n), np.arange(n + 1, dtype=np.int64) * d,
                         cols.astype(np.int32).ravel(), w.astype(np.float32).ravel())


@pytest.mark.parametrize("share", [0.0, 0.5, 0.85, 0.97])
def test_bins_of_few_and_many_columns(share):
    """20000 rows of 2500 products in one bin, none, half or most of them of
    rows in clusters (whose products still spread where a row of the cluster is
    a random one): every row is the oracle's, whichever kernel takes it."""
    n = 20000
    X = _rows_of(n, 50, 21, np.arange(int(share * n)) if share < 0.9 else
                 np.nonzero(synth.rng_for(1, 7).random(n) < share)[0])
    check_mcl_step(X, _run(X, r=2, prune=1e-4, topk=300), 2, 1e-4, 300)


@pytest.mark.parametrize("columns", [511, 512, 513])
def test_rows_of_one_bin_at_the_limit_of_columns(columns):
    """400 rows of 20 entries, each a row with the same `columns` columns (all
    empty rows): 10240 products on at most, or just more than, 512 columns."""
    rng = synth.rng_for(columns, 4)
    n, hubs = 2000, 30
    at = rng.permutation(n)
    hub, body, cols = at[:hubs], at[hubs:hubs + 400], np.sort(at[hubs + 400:hubs + 400 + columns])
    rows = [np.zeros(0, dtype=np.int64)] * n
    for v in hub:
        rows[v] = cols
    for v in body:
        rows[v] = np.sort(rng.choice(hub, size=20, replace=False))
    ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    v = 0.5 + 0.5 * rng.random(int(ip[-1]))
    lens = np.diff(ip)
    X = synth.HostCSR((n, n), ip, np.concatenate(rows).astype(np.int32),
                      (v / np.repeat(lens, lens)).astype(np.float32))
    got = _run(X, r=2, prune=0.0, topk=1000)
    assert set(np.diff(got.indptr)[body].tolist()) == {columns}
    check_mcl_step(X, got, 2, 0.0, 1000)
