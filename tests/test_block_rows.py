"""GPU parity of the rows of one block each: numbers of products at the edges
of the bins, more A entries than the block has threads (empty B rows among
them), repeats none, few, many, columns that cluster, one and three block
products.  Small-integer values: every partial sum is exact."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth
from helpers import assert_same_csr

pytestmark = pytest.mark.gpu

TARGETS = [1025, 1500, 2047, 2048, 2049, 3333, 4095, 4096, 4097, 6000, 8191, 8192, 8193]


def _operands(n, width, blen, seed, dtype):
    """B rows of 1..blen columns inside windows of `width` columns; A rows
    whose products number exactly TARGETS, some padded with 700 entries of
    empty B rows."""
    rng = synth.rng_for(seed, 3)
    kdim, empty = 9000, 800
    lens = rng.integers(1, blen + 1, size=kdim)
    lens[:2000] = 1
    lens[kdim - empty:] = 0
    start = rng.integers(0, n - width + 1) if width < n else 0
    cols = [np.sort(rng.choice(width, size=int(c), replace=False)) + start for c in lens]
    rows_a = []
    for target in TARGETS:
        for pad in (0, 700):
            order = rng.permutation(np.arange(2000, kdim - empty))
            upto = int(np.searchsorted(np.cumsum(lens[order]), target - 300))
            pick = order[:upto]
            rest = target - int(lens[pick].sum())
            pick = np.concatenate([pick, rng.choice(2000, size=rest, replace=False),
                                   rng.choice(empty, size=pad, replace=False) + kdim - empty])
            rows_a.append(rng.permutation(pick))

    def pack(rows, ncols, stream):
        ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
        col = np.concatenate(rows).astype(np.int32)
        return synth.HostCSR((len(rows), ncols), ip, col,
                             synth.draw_values(synth.rng_for(seed, stream), col.size, "int", dtype))

    return pack(rows_a, kdim, 4), pack(cols, n, 5)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,width,blen", [(6000, 6000, 60), (1 << 20, 1 << 20, 60),
                                          (1 << 20, 3000, 40), (1 << 24, 1 << 24, 20),
                                          ((1 << 24) + 1, (1 << 24) + 1, 25)])
@pytest.mark.parametrize("parts", [1, 3])
def test_rows_at_the_edges_of_the_bins(n, width, blen, parts, dtype):
    import torch  # brings up the HIP runtime that the library shares
    from paper_2603_21444_amd import binding
    assert torch.cuda.is_available()
    A, Bm = _operands(n, width, blen, 31 + blen, dtype)
    got_in = [(A, Bm)] if parts == 1 else synth.split_inner(A, Bm, np.array([0, 2500, 2600, 9000]))
    got = binding.batched([(binding.to_device(a), binding.to_device(b)) for a, b in got_in]).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), Bm.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True, what=f"n={n} width={width} parts={parts}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("width", [36, 50, 63, 64])
def test_rows_sorted_as_a_whole(width, dtype):
    """Rows of about width^2 products on few neighbouring columns, many or none
    of them repeated, with products past the last multiple of eight."""
    from paper_2603_21444_amd import binding
    rng = synth.rng_for(width, 11)
    n, k, m = 1 << 20, 70, 40
    rows = [np.sort(rng.choice(5000, size=width - t % 3, replace=False)) + 300000 for t in range(k)]
    rows += [np.arange(width - t % 3) + 700000 + width * t for t in range(k)]  # no repeats
    ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    B = synth.HostCSR((2 * k, n), ip, np.concatenate(rows).astype(np.int32),
                      rng.integers(-3, 4, size=ip[-1]).astype(dtype))
    pick = [h * k + rng.choice(k, size=width, replace=False) for h in (0, 1) for _ in range(m)]
    A = synth.HostCSR((2 * m, 2 * k), np.arange(2 * m + 1, dtype=np.int64) * width,
                      np.concatenate(pick).astype(np.int32),
                      rng.integers(-3, 4, size=2 * m * width).astype(dtype))
    got = binding.spgemm(binding.to_device(A), binding.to_device(B)).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), B.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True)
