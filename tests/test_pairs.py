"""GPU parity where B's columns and values are laid side by side (FP32, at
least twice as many A entries as B entries, B beyond an L2): aggregation
operators and short B rows, one and two block products, plain and as a
captured graph with other values on every replay."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth
from helpers import assert_same_csr

pytestmark = pytest.mark.gpu


def _inputs(kind, dtype):
    k = 600000
    A = synth.varnnz_csr(50000, k, 24, 56, 3, dtype, "int", stream=0)
    if kind == "aggregation":
        return A, synth.aggregation_csr(k, 5000, 3, dtype, "int")
    return A, synth.varnnz_csr(k, 70001, 0, 2, 3, dtype, "int", stream=1)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["aggregation", "short"])
@pytest.mark.parametrize("parts", [1, 2])
def test_short_rows_of_b(kind, parts, dtype):
    import torch  # brings up the HIP runtime that the library shares
    from paper_2603_21444_amd import binding
    from paper_2603_21444_amd.graph import StageGraph
    assert torch.cuda.is_available()
    A, Bm = _inputs(kind, dtype)
    blocks = [(A, Bm)] if parts == 1 else synth.split_inner(A, Bm, np.array([0, 200001, 600000]))
    ref, S = oracle.spgemm(A.astype(np.float64), Bm.astype(np.float64), with_abs=True)
    pairs = [(binding.to_device(a), binding.to_device(b)) for a, b in blocks]
    got = binding.batched(pairs).to_host()
    assert_same_csr(got, ref, S, dtype, exact=True, what="eager")
    graph = StageGraph(pairs)
    for t in (1, 2, 3):
        for _, b in pairs:
            b.vals.mul_(t)
        graph.replay()
        f = float(np.prod(np.arange(1, t + 1)))
        got = graph.result().to_host()
        scaled = synth.HostCSR(ref.shape, ref.indptr, ref.indices, ref.data * f)
        assert_same_csr(got, scaled, S * f, dtype, exact=True, what=f"replay {t}")
        x = torch.randn(1 << 18, device="cuda")
        float((x * x).sum())


def _wide(k, nc, hubs, dtype):
    """A: 50000 rows of 24..56 entries, the first `hubs` of them 30000; an
    aggregation operator to nc columns.  The words take nnz(B) / nc of the 256
    slots of the heavy rows, at most 32."""
    A = synth.varnnz_csr(50000, k, 24, 56, 3, dtype, "int", stream=0)
    rng = synth.rng_for(8, 3)
    lens = np.diff(A.indptr).astype(np.int64)
    lens[:hubs] = 30000
    cols = [np.sort(rng.choice(k, size=30000, replace=False)).astype(np.int32) for _ in range(hubs)]
    ip = np.concatenate([[0], np.cumsum(lens)])
    rest = A.indices[A.indptr[hubs]:]
    vals = np.concatenate([rng.integers(1, 4, size=30000 * hubs), A.data[A.indptr[hubs]:]])
    A = synth.HostCSR(A.shape, ip, np.concatenate(cols + [rest]).astype(np.int32), vals.astype(dtype))
    return A, synth.aggregation_csr(k, nc, 3, dtype, "int")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("hubs", [0, 5])
@pytest.mark.parametrize("nc", [18000, 20000, 60000])
def test_aggregation_and_heavy_rows_beside_the_words(nc, hubs, dtype):
    """Few enough entries of B per column for the words (18000: just too many,
    20000: nearly all of an eighth of the slots), without and with rows split
    over blocks, whose staging shares the region; eagerly, as a graph, and
    both types on one plan."""
    import torch
    from paper_2603_21444_amd import binding
    from paper_2603_21444_amd.graph import StageGraph
    assert torch.cuda.is_available()
    A, Bm = _wide(600000, nc, hubs, dtype)
    assert A.nnz >= 2 * Bm.nnz
    ref, S = oracle.spgemm(A.astype(np.float64), Bm.astype(np.float64), with_abs=True)
    pair = (binding.to_device(A), binding.to_device(Bm))
    plan = binding.Plan()
    for _ in range(2):
        assert_same_csr(binding.batched([pair], plan=plan).to_host(), ref, S, dtype, exact=True)
    other = np.float64 if dtype == np.float32 else np.float32
    oA, oB = binding.to_device(A.astype(other)), binding.to_device(Bm.astype(other))
    rp, nnz = plan.symbolic([oA], [oB])
    for a, b, t in ((oA, oB, other), (*pair, dtype)):
        col, vals = plan.numeric([a], [b], rp, nnz)
        got = binding.DeviceCSR(ref.shape, rp, col, vals).to_host()
        assert_same_csr(got, ref, S, t, exact=True)
    graph = StageGraph([pair])
    for _ in range(3):
        graph.replay()
        assert_same_csr(graph.result().to_host(), ref, S, dtype, exact=True)
        x = torch.randn(1 << 16, device="cuda")
        float((x * x).sum())
