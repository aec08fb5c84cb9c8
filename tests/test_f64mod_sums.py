"""Sums of up to four products of residues that are not centred with centred constants (the convolution's inner products), against 128-bit
integers: 4 q^2 / 2 is below the 2^101 that a chain of fused multiply-adds holds."""
import ctypes

import numpy as np
import pytest

from test_f64mod import PRIMES, lib, ptr  # noqa: F401  (lib: fixture)


@pytest.mark.parametrize("nd", [1, 4])
@pytest.mark.parametrize("q", PRIMES)
def test_sums_of_plain_residues(lib, q, nd):  # noqa: F811
    rng = np.random.default_rng(q % 999983 + nd)
    n = 50_000
    y = rng.integers(0, q, size=(n, nd), dtype=np.int64)
    y[:1000] = q - 1
    y[500:1000] -= rng.integers(0, 4, size=(500, nd)) % q
    half = [(q - 1) // 2, (q + 1) // 2]  # the centred constants of largest magnitude, of either sign
    for cw in ([half[0]] * nd, [half[1]] * nd, [half[a & 1] for a in range(nd)], rng.integers(0, q, size=nd).tolist()):
        cw = np.array(cw, dtype=np.uint64)
        r = np.empty(n, dtype=np.float64)
        assert lib.run_dot(ptr(y), ptr(cw), nd, ctypes.c_uint64(q), ptr(r), ctypes.c_size_t(n)) == 0
        bad = lib.chk_dot(ptr(y), ptr(cw), nd, ptr(r), ctypes.c_uint64(q), ctypes.c_size_t(n))
        assert bad < 0, f"q={q} nd={nd}: row {y[bad].tolist()} gave {r[bad]!r}"
