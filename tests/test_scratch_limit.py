"""Workspace sizes and the largest problem of the static scratch (what a
program that sizes its buffers once relies on), and split rows that find no
room for their segments."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import binding, synth
from helpers import assert_same_csr


@pytest.mark.parametrize("m,n,size", [(4096, 4096, 8622080), (1 << 18, 1 << 20, 2240974080),
                                      (100003, 120011, 252623104), (5, 1 << 23, 2190873344),
                                      (70000, 1000, 2754816), (1 << 20, (1 << 23) + 1, 2122589696)])
def test_workspace_sizes(m, n, size):
    assert binding.workspace_size(m, n, m) == size


@pytest.mark.gpu
def test_largest_problem_of_the_static_scratch():
    import torch
    n = 7225344  # one heavy row's region and descriptors: 2^27 bytes at most
    rng = synth.rng_for(3, 10)
    rows = np.sort(rng.choice(n, size=300, replace=False))
    ip = np.zeros(n + 1, dtype=np.int64)
    ip[rows + 1] = 20
    col = np.stack([rng.choice(rows, size=20, replace=False) for _ in rows]).astype(np.int32)
    A = synth.HostCSR((n, n), np.cumsum(ip), col.ravel(), rng.integers(-3, 4, size=6000).astype(np.float32))
    dA = binding.to_device(A)
    ref, S = oracle.spgemm(A.astype(np.float64), A.astype(np.float64), with_abs=True)
    plan = binding.Plan()
    rp = torch.empty(n + 1, dtype=torch.int32, device="cuda")
    plan.symbolic_noalloc([dA], [dA], rp, ref.nnz)
    c, v = plan.numeric([dA], [dA], rp, ref.nnz)
    assert plan.status() == binding.SPG_OK
    got = binding.DeviceCSR((n, n), rp, c, v).to_host()
    assert_same_csr(got, ref, S, np.float32, exact=True)
    big = binding.DeviceCSR((n + 1, n + 1), torch.zeros(n + 2, dtype=torch.int32, device="cuda"),
                            dA.col_idx[:0], dA.vals[:0])
    with pytest.raises(binding.SpgError) as e:
        plan.symbolic_noalloc([big], [big], torch.empty(n + 2, dtype=torch.int32, device="cuda"), 0)
    assert e.value.code == binding.SPG_ERR_SCRATCH


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_rows_without_room_for_their_segments(dtype):
    """Twelve rows that put 1026 products in every other range of 8192 columns
    and one in those between (128 segments each, one per 513 products) in a
    workspace of one heavy row: the last ones are not described."""
    n, k = 1 << 20, 65
    rng = synth.rng_for(4, 10)
    rows = [np.sort(rng.choice(8192, size=1026, replace=False)) + 16384 * f for f in range(64)]
    rows.append(np.arange(64) * 16384 + 8192 + rng.integers(0, 8192, size=64))
    ip = np.concatenate([[0], np.cumsum([r.size for r in rows])])
    B = synth.HostCSR((k, n), ip, np.concatenate(rows).astype(np.int32),
                      rng.integers(1, 5, size=ip[-1]).astype(dtype))
    A = synth.HostCSR((12, k), np.arange(13) * k, np.tile(np.arange(k), 12).astype(np.int32),
                      rng.integers(1, 5, size=12 * k).astype(dtype))
    t = binding.default_tuning()
    t.heavy_slots = 1
    plan = binding.Plan(tuning=t)
    got = binding.spgemm(binding.to_device(A), binding.to_device(B), plan=plan).to_host()
    assert plan.status() == binding.SPG_OK
    ref, S = oracle.spgemm(A.astype(np.float64), B.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True)
