"""The tuner's candidates, one per pair of kernels, and (GPU) products whose
columns are too many for the register sort, under every setting of the lanes:
the hash kernels of every group size, one row per wave, and the fallback."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import autotune, binding, synth
from helpers import assert_same_csr


@pytest.mark.parametrize("n", [1000, 1 << 20, 1 << 23, (1 << 24) + 1, 1 << 29])
def test_candidates_launch_different_kernels(n):
    t = binding.default_tuning()
    for b, cands in autotune.CANDIDATES.items():
        ds = autotune.distinct_candidates(b, n)
        assert ds[0] == (t.lanes[b], t.sub[b])
        launched = [autotune.kernels(b, lanes, min(sub, lanes), n) for lanes, sub in ds]
        assert len(set(launched)) == len(launched)
        for lanes, sub in cands:
            assert autotune.kernels(b, lanes, sub, n) in launched
    if n <= 1 << 20:
        assert [len(autotune.distinct_candidates(b, n)) for b in range(1, 12)] == \
            [2, 1, 1, 1, 2, 2, 3, 1, 1, 1, 1]


def _operands(n, dtype):
    A = synth.varnnz_csr(1500, 2000, 0, 60, 7, dtype, "int", stream=0)
    B = synth.varnnz_csr(2000, 3000, 0, 30, 7, dtype, "int", stream=1)
    rng = synth.rng_for(7, 2)
    spread = np.sort(rng.choice(n, size=3000, replace=False)).astype(np.int32)
    spread[:1500] = np.arange(1500) + n // 3  # half of the columns side by side
    spread = np.sort(np.unique(np.concatenate([spread, [0, n - 1]])))[:3000].astype(np.int32)
    return A, synth.HostCSR((2000, n), B.indptr, spread[B.indices % spread.size], B.data)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [(1 << 22) + 3, 1 << 24, (1 << 24) + 9, (1 << 28) + 77])
def test_more_columns_than_the_register_sort_takes(n, dtype):
    A, B = _operands(n, dtype)
    # the oracle on the columns in use, numbered
    used, inv = np.unique(B.indices, return_inverse=True)
    Bs = synth.HostCSR((B.shape[0], used.size), B.indptr, inv.astype(np.int32), B.data)
    ref, S = oracle.spgemm(A.astype(np.float64), Bs.astype(np.float64), with_abs=True)
    ref = synth.HostCSR((A.shape[0], n), ref.indptr, used[ref.indices].astype(np.int32), ref.data)
    dA, dB = binding.to_device(A), binding.to_device(B)
    seen = set()
    for lanes in (8, 16, 32, 64, 128, 512):
        for sub, window in ((4, 32), (16, 3), (64, 32)):
            t = binding.default_tuning()
            for b in range(1, 12):
                t.lanes[b], t.sub[b], t.sym_sub[b] = lanes, sub, sub
            t.max_window = window
            plan = binding.Plan(tuning=t)
            got = binding.spgemm(dA, dB, plan=plan).to_host()
            assert plan.status() == binding.SPG_OK
            seen |= {b for b, c in enumerate(plan.bins()[1]) if c}
            assert_same_csr(got, ref, S, dtype, exact=True, what=f"{lanes} lanes, sub {sub}")
    assert set(range(1, 8)) <= seen
