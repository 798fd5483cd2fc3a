"""GPU parity of row_ptr where one block scans the row counts and where three
kernels do: numbers of rows around whole threads, waves and the limit."""
import numpy as np
import pytest

import oracle
from paper_2603_21444_amd import synth
from helpers import assert_same_csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 63, 1023, 1024, 1025, 4097, 8191, 8192, 8193, 16385, 40000])
def test_row_ptr(m):
    import torch  # noqa: F401  (before the library)
    from paper_2603_21444_amd import binding
    rng = synth.rng_for(m, 1)
    k, n = 50, 300

    def csr(rows, cols, hi, stream):
        r = [np.sort(rng.choice(cols, size=int(c), replace=False))
             for c in rng.integers(0, hi, size=rows)]
        ip = np.concatenate([[0], np.cumsum([x.size for x in r])]).astype(np.int64)
        return synth.HostCSR((rows, cols), ip, np.concatenate(r).astype(np.int32),
                             synth.draw_values(synth.rng_for(m, stream), int(ip[-1]), "int",
                                               np.float32))

    A, B = csr(m, k, 4, 2), csr(k, n, 9, 3)
    got = binding.spgemm(binding.to_device(A), binding.to_device(B)).to_host()
    ref, S = oracle.spgemm(A.astype(np.float64), B.astype(np.float64), with_abs=True)
    assert_same_csr(got, ref, S, np.float32, exact=True, what=f"m={m}")
