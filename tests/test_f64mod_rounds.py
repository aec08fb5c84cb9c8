"""The rounds of the double-precision transforms (csrc/f64mod.h: where they reduce and where they do not) against exact integers
on the CPU: from inputs at the bound that the previous round leaves, in both signs and at random, with centred twiddles at
+-(q-1)/2, +-1, 0 and at random, every result is the right residue, every multiplicand stays below 4q (its quotient below
2^51) and every sum below 8q < 2^53, and what leaves the round is within the bound the next one assumes."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from workloads.params import CONFIGS, ntt_primes

HERE = os.path.dirname(os.path.abspath(__file__))
Q = [ntt_primes(16, 1)[0], CONFIGS["cfg5_resnet20_stage3"].params().moduli[11], ntt_primes(12, 1)[0], ntt_primes(12, 2, bits=20)[1]]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rounds") / "librounds.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "f64mod_rounds_check.cpp")],
                   check=True, capture_output=True, text=True)
    lib = ctypes.CDLL(so)
    lib.run_round.restype = ctypes.c_long
    lib.run_key_sum.restype = ctypes.c_long
    return lib


def operands(rng, q, low, high, n):
    """Eight values of [low, high] q per row (random, and rows of extremes in random signs), seven centred twiddles."""
    lo, hi = int(low * q), int(high * q)
    v = rng.integers(lo, hi + 1, size=(n, 8))
    edge = rng.random((n, 8)) < 0.5
    edge[: n // 4] = True
    v = np.where(edge, np.where(rng.random((n, 8)) < 0.5, lo, hi), v)
    h = (q - 1) // 2
    w = rng.integers(-h, h + 1, size=(n, 7))
    pick = rng.integers(0, 8, size=(n, 7))
    for k, c in enumerate((h, -h, 1, -1, 0)):
        w = np.where(pick == k, c, w)
    return v.astype(np.float64), w.astype(np.int64)


# name, stages, inverse, begin, end, bound of the inputs (low, high), bound of what leaves the round
ROUNDS = [
    ("hi pass, canonical residues", 3, 0, 0, 0, (0, 1), 3.13),
    ("hi pass, behind a conversion", 3, 0, 0, 0, (-0.5, 0.5), 2.42),
    ("forward round, from the widest hi pass", 3, 0, 1, 0, (-3.13, 3.13), 2.83),
    ("forward round, from another", 3, 0, 1, 0, (-2.83, 2.83), 2.78),
    ("last two forward stages", 2, 0, 0, 0, (-2.83, 2.83), 4.7),
    ("first two inverse stages, canonical residues", 2, 1, 0, 1, (0, 1), 1.26),
    ("first two inverse stages, a product", 2, 1, 0, 1, (-0.75, 0.75), 1.38),
    ("inverse round", 3, 1, 0, 1, (-1.46, 1.46), 1.46),
    ("inverse round, from two stages of the hi pass", 3, 1, 0, 0, (-1.73, 1.73), 3.8),
]


@pytest.mark.parametrize("value_only", [1, 0], ids=["value", "quotient"])
@pytest.mark.parametrize("name,stages,inverse,begin,end,bound,out", ROUNDS, ids=[r[0] for r in ROUNDS])
def test_rounds_are_exact_within_their_bounds(lib, name, stages, inverse, begin, end, bound, out, value_only):
    for k, q in enumerate(Q):
        rng = np.random.default_rng(100 + k)
        n = 60000
        v, w = operands(rng, q, *bound, n)
        worst = np.zeros(2)
        bad = lib.run_round(v.ctypes.data_as(ctypes.c_void_p), w.ctypes.data_as(ctypes.c_void_p), ctypes.c_uint64(q), stages, inverse, begin, end,
                            value_only, worst.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(n))
        slack = 16.0 / q                       # a reduced value may be one off q/2; eight of them add up
        assert bad == 0
        assert worst[0] <= 3.9 + slack and worst[1] < 8.0
        assert np.abs(v).max() / q <= out + slack, np.abs(v).max() / q


@pytest.mark.parametrize("digits,own", [(1, 1), (2, 0), (7, 3), (8, 8), (9, 7), (12, 12), (16, 8), (17, 15), (40, 0), (63, 31), (63, 63)])
def test_key_sums_of_any_number_of_digits(lib, digits, own):
    """The fused inner product's sum in a plain double, reduced where f64m_sum_due says: products of one sign whose residues lie around
    half the modulus, where their representatives are largest (up to 0.625 q), behind the digits two of multiplicands up to q.
    Unreduced, such a sum leaves 2^53 = 8q from about thirteen digits on."""
    for k, q in enumerate(Q[:3]):
        rng = np.random.default_rng(300 + k)
        n = 3000
        w = rng.integers(1, q, size=(n, digits + 2), dtype=np.uint64)
        target = (q // 2 + rng.integers(-q // 8, q // 8, size=w.shape)).tolist()
        y = np.array([[(t * pow(int(x), -1, q) + q // 2) % q - q // 2 for t, x in zip(tr, wr)] for tr, wr in zip(target, w)], dtype=np.float64)
        y[:, digits:] += np.where(y[:, digits:] < 0, q, 0)  # residues in [0, q): not reduced
        worst = np.zeros(1)
        assert lib.run_key_sum(y.ctypes.data_as(ctypes.c_void_p), w.ctypes.data_as(ctypes.c_void_p), ctypes.c_uint64(q), digits, own,
                               worst.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(n)) == 0
        assert worst[0] < 7.05  # q/2, eight of 0.625 q, two of 0.75 q, and some units
