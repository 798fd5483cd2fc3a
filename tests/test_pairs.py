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
