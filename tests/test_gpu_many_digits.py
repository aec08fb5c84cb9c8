"""GPU parity with as many digits as the moduli allow (one limb each): the inner product with the key is then a sum of up to 40
products, in double precision longer than one that stays below 2^53 unreduced."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2604_16834_amd as hx  # noqa: E402
from oracle import Oracle  # noqa: E402
from workloads import make_params  # noqa: E402
from gpu_common import rand_ct, rand_poly  # noqa: E402


def same(got, want):
    return bool(np.array_equal(hx.to_host(got), want))  # (a plain truth value: a failure prints no arrays)


@pytest.mark.parametrize("log_n,digits,level,bits", [(13, 40, 39, 50), (13, 21, 20, 50), (13, 12, 8, 50), (12, 40, 39, 50), (10, 21, 20, 50),
                                                     (13, 40, 39, 57), (10, 18, 17, 57)])
def test_inner_products_of_many_digits(log_n, digits, level, bits):
    """Key switch, rotations, product, merge and activation, bit for bit.  The switched polynomial is the constant -1, whose every
    digit is -1 at every point.  50-bit moduli: the key words lie just below half the modulus, all products of a sum have the
    same sign and the sum of 40 of them is 20 moduli, odd or even at random.  57-bit moduli: they lie just below the modulus, so that
    the residues' products are as large as they get (16 of them and P c0 meet before a reduction).  A uniform polynomial as well."""
    p = make_params(log_n, digits, 1, digits, bits=bits)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(6000 + digits + log_n + bits)
    key = np.empty((digits, 2, p.num_q + p.num_p, orc.N), dtype=np.uint64)
    for t, q in enumerate(p.moduli):
        key[:, :, t] = ((q - 1) // 2 if bits == 50 else q - 1) - rng.integers(0, 1 << 32, size=(digits, 2, orc.N), dtype=np.uint64)
    d_key = hx.from_host(key)
    load = lambda g: hx.ckks_key_load(ctx, d_key, g)
    one = np.ones((level + 1, orc.N), dtype=np.uint64)
    minus = np.stack([np.full(orc.N, q - 1, dtype=np.uint64) for q in p.moduli[:level + 1]])
    uniform = rand_ct(rng, p.moduli, level, orc.N)
    ct = np.stack([minus if bits > 50 else uniform[0], minus])
    d_ct = hx.from_host(ct)
    rlk = load(0)
    for c in (minus, uniform[1]):
        ok = same(hx.ckks_keyswitch(ctx, hx.from_host(c), level, rlk), orc.keyswitch(c, key, level))
        assert ok, "key switch"
    offs = [3, -1]
    dkeys = [load(hx.ckks_galois_element(ctx, r)) for r in offs]
    for hoisted in (False, True):
        outs = hx.ckks_rotate_hoisted(ctx, d_ct, level, offs, dkeys, hoisted)
        ok = [same(got, want) for got, want in zip(outs, orc.rotate_many(ct, level, offs, [key, key], hoisted))]
        assert all(ok), f"rotations, hoisted = {hoisted}"
    ok = same(hx.ckks_ctct_mul_relin(ctx, d_ct, d_ct, level, rlk), orc.ctct_mul_relin(ct, ct, key, level))
    assert ok, "product"
    sts = orc.n // 4
    blocks = [ct, np.stack([uniform[1], minus]), uniform]
    got = hx.he_accumulator_merge(ctx, [hx.from_host(b) for b in blocks], level, sts, hx.from_host(one),
                                  [None] + [load(hx.ckks_galois_element(ctx, -i * sts)) for i in (1, 2)])
    ok = same(got, orc.accumulator_merge(blocks, level, sts, one, {-sts: key, -2 * sts: key}))
    assert ok, "merge"
    k = (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
    (got,) = hx.he_poly_act_deg7(ctx, [d_ct], level, k, rlk, merged=True)
    ok = same(got, orc.poly_activation_merged(ct, level, k, key))
    assert ok, "activation"
