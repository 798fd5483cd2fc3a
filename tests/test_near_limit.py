"""GPU results for operands of nearly 2^31 entries: the last rows end where a
position plus a few lanes no longer fits 32 bits.  The other rows hold
entries without products, so that a call costs little more than reading A."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth
from helpers import assert_same_csr

pytestmark = pytest.mark.gpu

NNZ = 2 ** 31 - 1
K, N = 4096, 5000     # inner dimension and columns of the result
FIRST = 2048          # rows of B below are empty, the others hold one entry each


def _operand(tail):
    """Rows of 1024 entries on empty rows of B, then the rows `tail` (column
    lists): NNZ entries in all, values 1..7 by position."""
    import torch
    from paper_2603_21444_amd import binding
    t = sum(len(c) for c in tail)
    body = NNZ - t
    lens = np.full(-(-body // 1024), 1024, dtype=np.int64)
    lens[0] = body - 1024 * (lens.size - 1)
    rp = np.concatenate([[0], np.cumsum(np.concatenate([lens, [len(c) for c in tail]]))])
    col = torch.arange(NNZ, dtype=torch.int32, device="cuda")
    val = col.remainder(7).add_(1).float()
    col.remainder_(1024)
    col[body:] = torch.from_numpy(np.concatenate(tail).astype(np.int32)).cuda()
    A = binding.DeviceCSR((rp.size - 1, K), torch.from_numpy(rp.astype(np.int32)).cuda(), col, val)
    assert int(A.row_ptr[-1]) == NNZ
    last = synth.HostCSR((len(tail), K), rp[-len(tail) - 1:] - body,
                         np.concatenate(tail).astype(np.int32), val[body:].cpu().numpy())
    return A, last


def _one_entry_rows(first):
    """B: rows [0, first) empty, the others with one entry each."""
    k = np.arange(K - first)
    ip = np.concatenate([np.zeros(first, np.int64), np.arange(K - first + 1)])
    return synth.HostCSR((K, N), ip, (k * 37 % N).astype(np.int32),
                         (k % 5 + 1).astype(np.float32))


@pytest.mark.parametrize("length", [5, 250, 1024, 2000, 4000])
def test_row_keys(length):
    """No products at all, so only the row keys read A: rows counted by one
    thread, by a group and by a block."""
    from paper_2603_21444_amd import binding
    A, _ = _operand([np.arange(length)] * 3)
    B = binding.to_device(_one_entry_rows(K))
    plan = binding.Plan()
    rp, nnz = plan.symbolic([A], [B])
    assert nnz == 0 and plan.info() == (0, 0)
    assert int(rp.abs().max()) == 0
    bins, _ = plan.bins()
    assert bins[0] == A.shape[0]


def _check_tail(A, last, B, what):
    """C = A B with eager calls: rows before the last ones empty, the last
    ones the oracle's, exactly (small integers)."""
    from paper_2603_21444_amd import binding
    C = binding.spgemm(A, binding.to_device(B))
    t = last.shape[0]
    assert int(C.row_ptr[:-t].abs().max()) == 0
    got = binding.DeviceCSR((t, N), C.row_ptr[-t - 1:], C.col_idx, C.vals).to_host()
    ref, S = oracle.spgemm(last.astype(np.float64), B.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, np.float32, exact=True, what=what)


def _tail_row(products, length, rng):
    """`length` columns of which `products` (spread evenly, the last one among
    them) have an entry in B."""
    c = rng.permutation(FIRST)[:length]
    at = (np.arange(products) + 1) * length // products - 1
    c[at] = FIRST + rng.permutation(K - FIRST)[:products]
    return c


@pytest.mark.parametrize("length", [17, 100, 1023])
def test_rows_sorted_in_registers(length):
    """Rows of 1 to 1024 products, whose A entries take one chunk or many."""
    rng = synth.rng_for(length, 6)
    P = [p for p in (1, 9, 16, 17, 32, 50, 64, 100, 128, 200, 256, 500, 512, 900, 1023) if p <= length]
    A, last = _operand([_tail_row(p, length, rng) for p in P for _ in range(5)])
    _check_tail(A, last, _one_entry_rows(FIRST), f"rows of {length}")


def test_mcl_rows_on_few_columns():
    """X with 2^31 - 1 entries: nearly 2^21 rows of 1024 entries whose columns
    are empty rows of X, then rows of 257 to 1023 products on 300 columns."""
    import torch
    from mcl_check import check_mcl_step
    from paper_2603_21444_amd import binding
    n, half, ones = 1 << 22, (1 << 21) - 1000, 2048
    rng = synth.rng_for(1, 8)
    P = [257, 300, 512, 513, 700, 1000, 1023] * 3
    tail = []
    for p in P:  # p columns in [1024, 1024 + ones): rows of one entry each
        c = np.concatenate([rng.permutation(1024)[:1023 - p], 1024 + rng.permutation(ones)[:p]])
        tail.append(np.sort(c))
    tail[-1] = tail[-1][1:]
    body = NNZ - ones - sum(len(c) for c in tail)
    lens = np.zeros(n, dtype=np.int64)
    lens[1024:1024 + ones] = 1
    full = body // 1024
    lens[half:half + full] = 1024
    lens[half + full] = body - 1024 * full
    first = half + full + 1
    lens[first:first + len(P)] = [len(c) for c in tail]
    assert first + len(P) <= n - 300 and lens.sum() == NNZ
    rp = np.concatenate([[0], np.cumsum(lens)])
    col = torch.arange(NNZ, dtype=torch.int32, device="cuda")
    col[ones:ones + body].sub_(ones).remainder_(1024)
    one_col = (n - 300 + np.arange(ones) * 37 % 300).astype(np.int32)  # empty rows again
    col[:ones] = torch.from_numpy(one_col).cuda()
    col[ones + body:] = torch.from_numpy(np.concatenate(tail).astype(np.int32)).cuda()
    val = torch.full((NNZ,), 1.0 / 1024, dtype=torch.float32, device="cuda")
    w = (0.5 + rng.random(ones)).astype(np.float32)
    val[:ones] = torch.from_numpy(w).cuda()
    X = binding.DeviceCSR((n, n), torch.from_numpy(rp.astype(np.int32)).cuda(), col, val)
    plan = binding.Plan()
    got = binding.mcl_iteration(X, 2, 1e-4, 400, plan=plan, capacity=1 << 20)
    assert plan.status() == binding.SPG_OK
    del X, col, val
    small = np.zeros(n, dtype=np.int64)
    small[1024:1024 + ones] = 1
    small[first:first + len(P)] = [len(c) for c in tail]
    nt = sum(len(c) for c in tail)
    Xs = synth.HostCSR((n, n), np.concatenate([[0], np.cumsum(small)]),
                       np.concatenate([one_col, np.concatenate(tail)]).astype(np.int32),
                       np.concatenate([w, np.full(nt, 1.0 / 1024, np.float32)]).astype(np.float32))
    got = got.to_host()
    assert got.indptr[first] == 0
    assert check_mcl_step(Xs, got, 2, 1e-4, 400, rows=np.arange(first, first + len(P))) == 0


@pytest.mark.parametrize("lanes", [16, 1])
def test_as_many_rows_as_int32_counts(lanes):
    """2^31 - 1 rows of one product each, all in one row list: the register
    sort, and one thread per row."""
    import torch
    from paper_2603_21444_amd import binding
    m = NNZ
    rp = torch.arange(m + 1, dtype=torch.int64, device="cuda").int()
    col = torch.arange(m, dtype=torch.int32, device="cuda").remainder_(3)
    val = torch.arange(m, dtype=torch.int32, device="cuda").remainder_(7).float()
    A = binding.DeviceCSR((m, 3), rp, col, val)
    bcol, bval = (0, 5, 7), (2.0, 3.0, 5.0)
    B = binding.to_device(synth.HostCSR((3, 8), np.arange(4), np.array(bcol, np.int32),
                                        np.array(bval, np.float32)))
    t = binding.default_tuning()
    t.lanes[1] = lanes
    plan = binding.Plan(tuning=t)
    crp, nnz = plan.symbolic([A], [B])
    assert nnz == m and plan.info() == (m, m) and plan.bins()[0][1] == m
    ccol, cval = plan.numeric([A], [B], crp, nnz)
    assert plan.status() == binding.SPG_OK
    assert torch.equal(crp, rp)
    for k in range(3):  # row i holds the entry of B row i mod 3
        assert bool((ccol[k::3] == bcol[k]).all())
        assert torch.equal(cval[k::3], val[k::3] * bval[k])


def test_permute_nearly_2_31_rows():
    """2^31 - 1000 rows, all but the first and the last 600 empty, reversed."""
    import torch
    from paper_2603_21444_amd import binding
    m, n, k = 2 ** 31 - 1000, 5000, 600
    rng = synth.rng_for(2, 8)
    lens = rng.integers(0, 40, size=2 * k)
    cols = [rng.permutation(n)[:c].astype(np.int32) for c in lens]
    small = synth.HostCSR((2 * k, n), np.concatenate([[0], np.cumsum(lens)]), np.concatenate(cols),
                          rng.standard_normal(int(lens.sum())).astype(np.float32))
    rp = torch.full((m + 1,), int(small.indptr[k]), dtype=torch.int32, device="cuda")
    rp[:k + 1] = torch.from_numpy(small.indptr[:k + 1].astype(np.int32)).cuda()
    rp[m - k:] = torch.from_numpy(small.indptr[k:].astype(np.int32)).cuda()
    A = binding.DeviceCSR((m, n), rp, torch.from_numpy(small.indices).cuda(),
                          torch.from_numpy(small.data).cuda())
    q = synth.random_permutation(n, 4)
    p = torch.arange(m, dtype=torch.int32, device="cuda").neg_().add_(m - 1)
    plan = binding.Plan()
    B = binding.permute(A, p, torch.from_numpy(q.astype(np.int32)).cuda(), plan=plan)
    assert plan.status() == binding.SPG_OK
    ref = oracle.permute(small.astype(np.float64), np.arange(2 * k)[::-1].copy(), q)
    ip = torch.from_numpy(ref.indptr.astype(np.int32)).cuda()
    assert torch.equal(B.row_ptr[:k + 1], ip[:k + 1]) and torch.equal(B.row_ptr[m - k:], ip[k:])
    assert bool((B.row_ptr[k:m - k + 1] == ip[k]).all())
    assert np.array_equal(B.col_idx.cpu().numpy(), ref.indices)
    assert np.array_equal(B.vals.cpu().numpy().astype(np.float64), ref.data)
