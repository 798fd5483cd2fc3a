"""GPU permutation of rows at the edges of the length classes, few and many
rows of each, columns repeated in no row, against the oracle bit for bit; and
arrays that are no permutations in ways a plain store could hide."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _torch_first():
    import torch  # brings up the HIP runtime that the library shares
    assert torch.cuda.is_available()


def _dev(p):
    import torch
    return torch.from_numpy(np.ascontiguousarray(p, dtype=np.int32)).cuda()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("lens", [[0, 1, 15, 16, 17], [63, 64, 65, 255, 256, 257],
                                  [4095, 4096, 4097, 3], [16] * 1025, [5]])
def test_rows_at_class_edges(lens, dtype):
    from paper_2603_21444_amd import binding
    n = 6000
    rng = synth.rng_for(5, len(lens))
    cols = [rng.choice(n, size=c, replace=False).astype(np.int32) for c in lens]
    A = synth.HostCSR((len(lens), n), np.concatenate([[0], np.cumsum(lens)]).astype(np.int64),
                      np.concatenate(cols), rng.standard_normal(sum(lens)).astype(dtype))
    p, q = synth.random_permutation(len(lens), 3), synth.random_permutation(n, 4)
    plan = binding.Plan()
    got = binding.permute(binding.to_device(A), _dev(p), _dev(q), plan=plan)
    assert plan.status() == binding.SPG_OK
    h, ref = got.to_host(), oracle.permute(A.astype(np.float64), p, q)
    assert np.array_equal(h.indptr, ref.indptr)
    assert np.array_equal(h.indices, ref.indices)
    assert np.array_equal(h.data.astype(np.float64), ref.data)


@pytest.mark.parametrize("where", ["rows", "columns", "both"])
@pytest.mark.parametrize("bad", [(0, 1), (7, -1), (2, 300)])
def test_no_permutation_after_a_good_one(where, bad):
    """The inverse of an earlier call is still in the workspace: a repeated,
    negative or too large index is found all the same."""
    import torch
    from paper_2603_21444_amd import binding
    n = 300
    A = binding.to_device(synth.varnnz_csr(n, n, 1, 9, 6, np.float32, "normal"))
    good = np.arange(n, dtype=np.int32)[::-1].copy()
    p = good.copy()
    p[bad[0]] = p[bad[1]] if bad[1] == 1 else bad[1]
    plan = binding.Plan()
    binding.permute(A, _dev(good), _dev(good), plan=plan)
    assert plan.status() == binding.SPG_OK
    d = _dev(p)
    rows, cols = (d if where != "columns" else _dev(good)), (d if where != "rows" else _dev(good))
    out = (torch.full((n + 1,), -7, dtype=torch.int32, device="cuda"),
           torch.full((A.nnz,), -7, dtype=torch.int32, device="cuda"),
           torch.full((A.nnz,), -7.0, device="cuda"))
    binding.permute(A, rows, cols, plan=plan, out=out)
    assert plan.status() == binding.SPG_ERR_INVALID
    assert all(bool((t == -7).all()) for t in out)


@pytest.mark.parametrize("lens", [[255, 256, 257, 258], [511, 512, 513, 767, 768, 769],
                                  [1023, 1024, 1025], [2047, 2048, 2049, 3072, 3073],
                                  [4096, 4097, 5999, 1025, 0, 300, 4098, 2000, 64, 70] * 30,
                                  [257, 1024, 100, 16] * 700])
def test_rows_of_the_longer_classes(lens):
    """Rows of 65 to 4096 entries and longer at the numbers of entries that a
    wave or a lane starts to hold, few and more of them than blocks."""
    test_rows_at_class_edges(lens, np.float32)
