"""GPU parity of the register-sorted rows: rows whose number of products sits
at the edges of every bin, over B rows of uneven length (empty ones among
them), columns that repeat a lot or never, columns at the limits of the key,
one and two block products.  Small-integer values: every partial sum is
exact, so the values must be equal."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth
from helpers import assert_same_csr

pytestmark = pytest.mark.gpu

EDGES = [16, 32, 64, 128, 256, 512, 1024]


def _operands(n, dtype, seed, blen):
    """A and B with rows of 1, edge - 1, edge and edge + 1 products, the
    entries of half the rows padded with up to 150 entries of empty B rows."""
    rng = synth.rng_for(seed, 3)
    kdim = 4000
    lens = rng.integers(1, blen + 1, size=kdim)
    lens[:blen] = 1
    lens[kdim - 200:] = 0
    lens = np.minimum(lens, n)
    rows_b = [np.sort(rng.choice(n, size=int(c), replace=False)) if n < 5000 else
              np.unique(rng.integers(0, n, size=int(c))) for c in lens]
    rows_b[5] = np.array([n - 1])
    rows_b[6] = np.array([0])
    lens = np.array([r.size for r in rows_b])
    ones = np.flatnonzero(lens == 1)
    rows_a = []
    for e in EDGES:
        for target in (1, e - 1, e, e + 1):
            for pad in (0, int(rng.integers(1, 150))):
                pick, total = [], 0
                for r in rng.permutation(kdim - 200):
                    if r not in (5, 6) and total + lens[r] <= target - 2:
                        pick.append(r)
                        total += lens[r]
                    if total == target - 2:
                        break
                pool = [r for r in ones if r not in set(pick)]
                pick += pool[:target - total]
                pick += list(range(kdim - 200, kdim - 200 + pad))
                rows_a.append(rng.permutation(np.array(pick)))

    def pack(rows, ncols, stream):
        ip = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
        col = np.concatenate(rows).astype(np.int32)
        return synth.HostCSR((len(rows), ncols), ip, col,
                             synth.draw_values(synth.rng_for(seed, stream), col.size, "int", dtype))

    return pack(rows_a, kdim, 4), pack(rows_b, n, 5)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,blen", [(40, 16), (3000, 17), (1 << 22, 33), ((1 << 22) + 1, 5),
                                    ((1 << 24) + 1, 7), ((1 << 25) + 1, 3)])
def test_rows_at_the_edges_of_the_bins(n, blen, dtype):
    from paper_2603_21444_amd import binding
    A, Bm = _operands(n, dtype, 17 + blen, blen)
    got = binding.spgemm(binding.to_device(A), binding.to_device(Bm)).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), Bm.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True, what=f"n={n}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_rows_of_two_block_products(dtype):
    from paper_2603_21444_amd import binding
    A, Bm = _operands(2500, dtype, 29, 19)
    parts = synth.split_inner(A, Bm, np.array([0, 1700, 4000]))
    got = binding.batched([(binding.to_device(a), binding.to_device(b)) for a, b in parts]).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), Bm.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, dtype, exact=True, what="two blocks")
