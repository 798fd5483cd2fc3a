"""GPU parity of the rows split over many blocks: products on few and on many
columns (places from a dense panel, a bitmap, buckets), with many and with few
repeats, more A entries than a window has threads, B rows of more than 2^20
entries, one and several block products.  Small-integer values: every partial
sum is exact, so the values must be equal."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth
from helpers import assert_same_csr

pytestmark = pytest.mark.gpu


def _csr(rows, ncols, seed, stream, dtype):
    ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    return synth.HostCSR((len(rows), ncols), ip, col,
                         synth.draw_values(synth.rng_for(seed, stream), col.size, "int", dtype))


def _operands(n, dtype, seed):
    rng = synth.rng_for(seed, 1)
    kdim = 6000

    def cols(lo, hi, size):
        size = min(size, hi - lo)
        if hi - lo <= 1 << 16:
            return np.sort(rng.choice(np.arange(lo, hi), size=size, replace=False))
        return np.unique(rng.integers(lo, hi, size=size))

    B = [cols(0, n, int(c)) for c in rng.integers(1, 33, size=kdim)]
    for r in range(50):                      # a narrow band: many repeats
        B[r] = cols(n // 3, n // 3 + 9000, 3000) if n > 30000 else cols(0, n, 300)
    for r in range(50, 60):                  # most of one range of 8192 columns
        B[r] = cols(0, min(n, 8192), 6000)
    B[60] = cols(0, n, n // 2 + 7)           # a long row
    for r in range(61, 4000, 3):             # empty rows
        B[r] = B[r][:0]
    # the first and the last column
    B[4000], B[4001] = np.array([0]), np.array([n - 1])
    rest = np.arange(4000, kdim)
    A = [np.array([60]), np.arange(50, 60), np.arange(50), np.arange(50, 61), rest, rest[:500],
         np.arange(kdim), np.concatenate([np.arange(20, 24), rest[:300]]), rest[:230], rest[:260],
         np.array([], dtype=np.int64), np.array([4000, 4001]), rest[:249], rest[:900]]
    return (_csr([rng.permutation(a) for a in A], kdim, seed, 2, dtype),
            _csr(B, n, seed, 3, dtype))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [9000, (1 << 18) + 5, (1 << 20) + 1, (1 << 21) + 77, 1 << 23])
def test_split_rows(n, dtype):
    from paper_2603_21444_amd import binding
    A, B = _operands(n, dtype, 5)
    got = binding.spgemm(binding.to_device(A), binding.to_device(B)).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), B.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True, what=f"n={n}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_split_rows_of_block_products(dtype):
    from paper_2603_21444_amd import binding
    A, B = _operands(1 << 20, dtype, 6)
    parts = synth.split_inner(A, B, np.array([0, 55, 61, 4100, 6000]))
    got = binding.batched([(binding.to_device(a), binding.to_device(b)) for a, b in parts]).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), B.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True, what="four blocks")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [(1 << 17) - 3, 1 << 17, (1 << 17) + 9, (1 << 18) - 1, 3 << 17])
def test_split_rows_about_the_spans_of_the_bitmap(n, dtype):
    """Segments of up to, and just more than, 2^17 (FP64) and 2^18 columns."""
    test_split_rows(n, dtype)
