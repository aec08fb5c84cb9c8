"""GPU parity at the sizes where the launch rules change: how many batch items a lo-pass workgroup takes, which kernel takes the
layer's multiply-accumulate, how many digits a decomposition launches at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2604_16834_amd as hx  # noqa: E402
from oracle import Oracle  # noqa: E402
from workloads import conv_tap_offsets, make_params  # noqa: E402
from gpu_common import rand_ct, rand_poly, w_residues  # noqa: E402
from test_gpu_parity import fc_case  # noqa: E402


@pytest.mark.parametrize("batch,bits", [(95, 50), (191, 50), (192, 57), (193, 50), (289, 50), (289, 57), (769, 50), (769, 57)])
def test_ntt_items_per_workgroup(batch, bits):
    """Two limbs of four slices at N = 2^13: one item per workgroup below 192 polynomials, two from there (the inverse pass' most; a
    workgroup of one at 193), three at 289 with a ragged last share, eight (the forward pass' most) at 769, where a few
    workgroups get seven."""
    p = make_params(13, 2, 1, 1, bits=bits)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(2000 + batch)
    idx = [2, 1]
    polys = np.stack([rand_poly(rng, [p.moduli[t] for t in idx], orc.N) for _ in range(batch)])
    d = hx.from_host(polys)
    hx.ckks_ntt_fwd(ctx, d, idx)
    assert np.array_equal(hx.to_host(d), orc.ntt_many(polys, idx))
    hx.ckks_ntt_inv(ctx, d, idx)
    assert np.array_equal(hx.to_host(d), polys)


def random_conv(log_n, c_in, c_out, bits_of_weights=31, seed=1):
    """A convolution of uniform residues: (oracle's outputs, the device's outputs) in the default schedule."""
    p = make_params(log_n, 3, 2, 2)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(3000 + seed)
    level = p.num_q - 1
    q = p.moduli
    cts = [rand_ct(rng, q, level, orc.N) for _ in range(c_in)]
    offs = conv_tap_offsets(4)
    keys = {o: np.stack([np.stack([rand_poly(rng, q, orc.N) for _ in range(2)]) for _ in range(p.dnum)]) for o in offs if o}
    masks = np.stack([rand_poly(rng, q[:level + 1], orc.N) for _ in range(9)])
    w = rng.integers(-2 ** bits_of_weights, 2 ** bits_of_weights, size=(c_out, c_in, 9))
    w[0, 0, :2] = (2 ** bits_of_weights - 1, -2 ** bits_of_weights + 1)
    want = orc.he_conv(cts, level, 4, keys, masks, w)
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(keys[o]), hx.ckks_galois_element(ctx, o)) if o else None for o in offs]
    outs = hx.he_conv_batched(ctx, 4, 4, 2, level, [hx.from_host(c) for c in cts], dkeys, hx.from_host(masks),
                              hx.from_host(w_residues(w, q, level)), c_out, weight_bits=hx.conv_weight_bits(w))
    return want, [hx.to_host(o) for o in outs]


@pytest.mark.parametrize("log_n,c_in,c_out,bits", [(6, 2, 3, 48), (12, 1, 1, 31), (12, 3, 5, 48), (12, 29, 2, 31), (12, 15, 8, 22),
                                                   (12, 3, 33, 48), (12, 3, 64, 48), (14, 1, 9, 31)])
def test_weighted_sum_kernels(log_n, c_in, c_out, bits):
    """Both sides of the rule: the double-precision kernel with one to eight outputs per thread, a ragged chunk of eight terms,
    more terms than one stage of weights (261), a column block beyond the ring (N = 2^6) and several groups of outputs; the
    matrix-core kernel with a ragged block of terms (27 x 64 outputs).  Exact, for weights up to the modulus' size."""
    want, got = random_conv(log_n, c_in, c_out, bits, seed=c_in * 100 + c_out)
    for o in range(c_out):
        assert np.array_equal(got[o], want[o]), f"output {o}"


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level", [(15, 5, 2, 3, 4), (15, 13, 8, 2, 12), (15, 12, 9, 2, 7), (15, 11, 11, 1, 10),
                                                          (15, 14, 14, 1, 13), (15, 12, 12, 1, 6), (15, 12, 10, 1, 9),
                                                          (16, 7, 3, 4, 5), (13, 7, 12, 3, 6)])
def test_digits_together(log_n, num_q, num_p, dnum, level):
    """All digits of a small decomposition in one launch: ragged last digits (1 of 2, 6 of 7, 2 of 6 limbs) and a single digit, rows of
    4, 8 and 16 conversion constants on both sides (7 to 14 real ones of sixteen), target counts that are not multiples of
    four, with the inner product inside the second pass (key switch) and behind it (hoisted rotations)."""
    p = make_params(log_n, num_q, num_p, dnum)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(4000 + num_q)
    ct = rand_ct(rng, p.moduli, level, orc.N)
    offs = [3, -1]
    keys = [np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(dnum)]) for _ in offs]
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(k), hx.ckks_galois_element(ctx, r)) for k, r in zip(keys, offs)]
    out = hx.ckks_keyswitch(ctx, hx.from_host(ct[1]), level, dkeys[0])
    assert np.array_equal(hx.to_host(out), orc.keyswitch(ct[1], keys[0], level))
    outs = hx.ckks_rotate_hoisted(ctx, hx.from_host(ct), level, offs, dkeys, True)
    for got, want in zip(outs, orc.rotate_many(ct, level, offs, keys, True)):
        assert np.array_equal(hx.to_host(got), want)


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level", [(12, 7, 3, 3, 6), (12, 5, 5, 1, 4), (13, 9, 2, 5, 7), (13, 9, 2, 5, 8), (15, 11, 4, 3, 8),
                                                          (16, 6, 2, 3, 3), (16, 10, 3, 4, 9)])
def test_integer_digits_together(log_n, num_q, num_p, dnum, level):
    """All digits of a decomposition in one launch per pass with 57-bit moduli: ragged last digits (1 of 3, 1 of 2, 1 of 4 limbs), a single
    digit, five digits (more than the kernel that keeps its key words takes) and four of five, two of three; one, two and eight
    polynomials (unhoisted rotations), and hoisted ones; at N = 2^16 with ten limbs a workgroup of the second pass takes two
    rows (polynomial, digit) for one polynomial and four for two, stepping past each digit's own limbs."""
    p = make_params(log_n, num_q, num_p, dnum, bits=57)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(5000 + num_q)
    ct = rand_ct(rng, p.moduli, level, orc.N)
    offs = [1, -2, 3, 4, -5, 6, 7, -8][: 8 if log_n <= 12 else 2]
    keys = [np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(dnum)]) for _ in offs]
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(k), hx.ckks_galois_element(ctx, r)) for k, r in zip(keys, offs)]
    out = hx.ckks_keyswitch(ctx, hx.from_host(ct[1]), level, dkeys[0])
    assert np.array_equal(hx.to_host(out), orc.keyswitch(ct[1], keys[0], level))
    for hoisted in (False, True):
        outs = hx.ckks_rotate_hoisted(ctx, hx.from_host(ct), level, offs, dkeys, hoisted)
        for got, want in zip(outs, orc.rotate_many(ct, level, offs, keys, hoisted)):
            assert np.array_equal(hx.to_host(got), want)


@pytest.mark.parametrize("num_p", [9, 10, 11])
def test_merged_divisions_of_many_special_primes(num_p):
    """Ten, eleven and twelve dropped limbs at N = 2^15 (rows of twelve conversion constants): the merged activation's divisions by
    P q_level, down to two remaining limbs."""
    p = make_params(15, 5, num_p, 1)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(4500 + num_p)
    level, k = 4, (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
    ct = rand_ct(rng, p.moduli, level, orc.N)
    key = np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)])])
    (got,) = hx.he_poly_act_deg7(ctx, [hx.from_host(ct)], level, k, hx.ckks_key_load(ctx, hx.from_host(key), 0), merged=True)
    assert np.array_equal(hx.to_host(got), orc.poly_activation_merged(ct, level, k, key))


@pytest.mark.parametrize("log_n,num_p,dnum", [(11, 2, 3), (12, 2, 3), (13, 2, 3), (13, 1, 6)])
def test_integer_merge_layer_and_layout(log_n, num_p, dnum):
    """What adds P c0 to its inner products or sums in its divisions' last step, with 57-bit moduli: the merge of four blocks, the fully
    connected layer (three outputs, a ragged block of second rotations) and the layout in both schedules; up to three digits,
    whose key words a thread keeps, and six."""
    p = make_params(log_n, 6, num_p, dnum, bits=57)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(5500 + log_n + dnum)
    level, q, n = p.num_q - 1, p.moduli, orc.N
    pt = lambda lv: rand_poly(rng, q[:lv + 1], n)
    ext = lambda lv: rand_poly(rng, [q[t] for t in orc.ext_moduli_idx(lv)], n)
    keys, dkeys = {}, {}

    def key(r):
        if r % orc.n == 0:
            return None
        if r not in keys:
            keys[r] = np.stack([np.stack([rand_poly(rng, q, n) for _ in range(2)]) for _ in range(dnum)])
            dkeys[r] = hx.ckks_key_load(ctx, hx.from_host(keys[r]), hx.ckks_galois_element(ctx, r))
        return dkeys[r]

    same = lambda got, want: bool(np.array_equal(hx.to_host(got), want))
    cts = [rand_ct(rng, q, level, n) for _ in range(4)]
    d_cts = [hx.from_host(c) for c in cts]
    sts, mask = orc.n // 4, pt(level)
    got = hx.he_accumulator_merge(ctx, d_cts, level, sts, hx.from_host(mask), [key(-i * sts) for i in range(4)])
    ok = same(got, orc.accumulator_merge(cts, level, sts, mask, keys))
    assert ok, "merge"
    d_in, d_out, batch, base = 8, 3, 5, 2
    _, lo, hi = orc.fc_shifts(d_in, d_out, batch, base)
    ops = (np.stack([pt(level) for _ in range(d_out)]), pt(level - 1), np.stack([pt(level - 2) for _ in range(batch)]), pt(level - 3))
    got = hx.he_fc_batched(ctx, d_cts[0], level, d_in, d_out, batch, base, *[hx.from_host(o) for o in ops], [key(1 << s) for s in range(3)],
                           [key(-i) for i in range(d_out)], [key(r) for r in lo], [key(r) for r in hi])
    ok = same(got, orc.fc_batched(cts[0], level, d_in, d_out, batch, base, *ops, keys))
    assert ok, "fully connected layer"
    lo, hi = [0, 3, 5], [7, 0]
    for schedule in (hx.HE_RELAYOUT_DIRECT, hx.HE_RELAYOUT_DEFERRED):
        deferred = schedule == hx.HE_RELAYOUT_DEFERRED
        masks = [[(ext if deferred else pt)(level) for _ in lo] for _ in hi]
        masks[1][2] = None
        outs = hx.he_relayout_two_rotations(ctx, d_cts[:3], level, lo, [key(r) for r in lo], hi, [key(r) for r in hi],
                                            [[None if m is None else hx.from_host(m) for m in row] for row in masks], schedule=schedule)
        oracle = orc.relayout_two_rotations_deferred if deferred else orc.relayout_two_rotations
        ok = [same(o, oracle(c, level, lo, hi, masks, keys)) for o, c in zip(outs, cts)]
        assert all(ok), f"layout, schedule {schedule}"


@pytest.mark.parametrize("batch,base", [(38, 3), (40, 36)])
def test_masked_sums_of_the_layout(batch, base):
    """More second rotations than one launch of the masked sums takes (13 = 12 + 1, the last sum without its third mask), and more
    first rotations than one launch takes (36 = 32 + 4) with a sum that has masks for four of them only."""
    k = fc_case(8, 1, batch, base, seed=700 + batch)
    assert np.array_equal(hx.to_host(k["run"]()), k["want"])


@pytest.mark.parametrize("bits,dnum,level", [(50, 3, 6), (50, 1, 6), (50, 7, 3), (57, 3, 5)])
def test_whole_ring_kernels(bits, dnum, level):
    """The one-workgroup transforms of N = 2^12, both arithmetics: in place and from a list, batches and any order of moduli, the rescale in
    one launch; and what goes pass by pass there with the double-precision arithmetic (with the integer one the whole-ring kernels take the
    transforms): conversions of digits of three (ragged), seven and one limbs, divisions without operands (key switch) and
    with an addend (unhoisted rotation).  The divisions of the double-precision whole-ring kernels: test_whole_ring_divisions."""
    p = make_params(12, 7, 7 if dnum == 1 else 3, dnum, bits=bits)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(5000 + bits + dnum)
    idx = [p.num_q, 0, 6, 3, 1]
    polys = np.stack([rand_poly(rng, [p.moduli[t] for t in idx], orc.N) for _ in range(3)])
    polys[0, :, :2] = [[0, p.moduli[t] - 1] for t in idx]
    d = hx.from_host(polys)
    hx.ckks_ntt_fwd(ctx, d, idx)
    assert np.array_equal(hx.to_host(d), orc.ntt_many(polys, idx))
    hx.ckks_ntt_inv(ctx, d, idx)
    assert np.array_equal(hx.to_host(d), polys)
    ct = rand_ct(rng, p.moduli, level, orc.N)
    offs = [5, -2]
    keys = [np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(dnum)]) for _ in offs]
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(k), hx.ckks_galois_element(ctx, r)) for k, r in zip(keys, offs)]
    d_ct = hx.from_host(ct)
    assert np.array_equal(hx.to_host(hx.ckks_keyswitch(ctx, hx.from_host(ct[1]), level, dkeys[0])), orc.keyswitch(ct[1], keys[0], level))
    assert np.array_equal(hx.to_host(hx.ckks_rescale(ctx, d_ct, level)), orc.rescale(ct, level))
    for hoisted in (True, False):
        outs = hx.ckks_rotate_hoisted(ctx, d_ct, level, offs, dkeys, hoisted)
        for got, want in zip(outs, orc.rotate_many(ct, level, offs, keys, hoisted)):
            assert np.array_equal(hx.to_host(got), want)


@pytest.mark.parametrize("num_p", [3, 6, 8, 10, 14])
def test_whole_ring_divisions(num_p):
    """N = 2^12: divisions of whole sums into 113 to 256 limb-polys are one launch each way.  Six hoisted rotations of six digits (with up to four, whose
    inner products go on into the inverse transform, they take no such division: two digits), the eight of a direct convolution
    and the merged divisions of a deferred one, by three to fourteen special primes (four, eight and sixteen terms) and with the
    level's own limb (four, eight, nine and twelve of twelve, sixteen)."""
    p = make_params(12, 12, num_p, 2)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(5200 + num_p)
    level, q, n = p.num_q - 1, p.moduli, orc.N
    n_rot, c_out = 6, 6
    assert all(112 < rows <= 256 for rows in ((level + 1) * 2 * n_rot, (level + 1) * 2 * 8, level * 2 * c_out))  # ntt_mid_moddown's window
    ct = rand_ct(rng, q, level, n)
    toffs = conv_tap_offsets(4)
    offs = [o for o in toffs if o][:n_rot]
    keys = {o: np.stack([np.stack([rand_poly(rng, q, n) for _ in range(2)]) for _ in range(p.dnum)]) for o in toffs if o}
    dkeys = {o: hx.ckks_key_load(ctx, hx.from_host(k), hx.ckks_galois_element(ctx, o)) for o, k in keys.items()}
    outs = hx.ckks_rotate_hoisted(ctx, hx.from_host(ct), level, offs, [dkeys[o] for o in offs], True)
    for out, want in zip(outs, orc.rotate_many(ct, level, offs, [keys[o] for o in offs], True)):
        assert np.array_equal(hx.to_host(out), want), "rotations"
    p6 = make_params(12, 12, num_p, 6)
    orc6, ctx6 = Oracle(p6), hx.Context(p6)
    keys6 = [np.stack([np.stack([rand_poly(rng, p6.moduli, n) for _ in range(2)]) for _ in range(6)]) for _ in offs]
    outs = hx.ckks_rotate_hoisted(ctx6, hx.from_host(ct), level, offs, [hx.ckks_key_load(ctx6, hx.from_host(k), hx.ckks_galois_element(ctx6, o)) for k, o in zip(keys6, offs)], True)
    for out, want in zip(outs, orc6.rotate_many(ct, level, offs, keys6, True)):
        assert np.array_equal(hx.to_host(out), want), "rotations of six digits"
    w = rng.integers(-2 ** 31, 2 ** 31, size=(c_out, 1, 9))
    for al in (hx.HE_CONV_ALIGN_DIRECT, hx.HE_CONV_DEFERRED_MERGED):
        idx = orc.ext_moduli_idx(level) if al == hx.HE_CONV_DEFERRED_MERGED else list(range(level + 1))
        masks = np.stack([rand_poly(rng, [q[t] for t in idx], n) for _ in range(9)])
        w_res = w_residues(w, [q[t] for t in idx], len(idx) - 1)
        want = orc.he_conv_deferred([ct], level, 4, keys, masks, w, merged=True) if al == hx.HE_CONV_DEFERRED_MERGED else orc.he_conv([ct], level, 4, keys, masks, w)
        outs = hx.he_conv_batched(ctx, 4, 4, 2, level, [hx.from_host(ct)], [dkeys.get(o) for o in toffs], hx.from_host(masks), hx.from_host(w_res), c_out, alignment=al)
        assert all(np.array_equal(hx.to_host(o), want[i]) for i, o in enumerate(outs)), f"convolution, schedule {al}"


@pytest.mark.parametrize("log_n,bits,stored", [(14, 50, False), (13, 50, False), (12, 50, False), (11, 50, True), (13, 57, True)])
def test_products_stay_within_their_workspace(log_n, bits, stored):
    """The scratch of a product is a key switch's, plus the tensor product's three polynomials only where a kernel stores them; product
    and activation (two batches in flight, or with merged divisions on the double-precision rings up to 2^13 all nine together) with exactly
    the queried bytes give the oracle's residues and touch nothing around them."""
    p = make_params(log_n, 6, 2, 3, bits=bits)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(7000 + log_n + bits)
    level, n_ct = p.num_q - 1, 9
    key = np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(p.dnum)])
    rlk = hx.ckks_key_load(ctx, hx.from_host(key), 0)
    product = hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_CTCT_MUL_RELIN, level)
    assert product == hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_KEYSWITCH, level) + (3 * (level + 1) * orc.N * 8 if stored else 0)

    def guarded(nbytes):
        buf = torch.full((nbytes // 8 + 128,), 0x5A5A5A5A, dtype=torch.int64, device="cuda")
        return buf, buf[64:-64]

    def untouched(buf):
        return bool((buf[:64] == 0x5A5A5A5A).all()) and bool((buf[-64:] == 0x5A5A5A5A).all())

    cts = [rand_ct(rng, p.moduli, level, orc.N) for _ in range(2)]
    d_cts = [hx.from_host(c) for c in cts]
    buf, ws = guarded(product)
    ok = np.array_equal(hx.to_host(hx.ckks_ctct_mul_relin(ctx, d_cts[0], d_cts[1], level, rlk, ws=ws)), orc.ctct_mul_relin(*cts, key, level))
    assert ok and untouched(buf)
    k = (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
    want = {True: [orc.poly_activation_merged(c, level, k, key) for c in cts], False: [orc.poly_activation(c, level, k, key) for c in cts]}
    for merged in (True, False):
        buf, ws = guarded(hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_POLY_ACT, level, n_ct))
        outs = hx.he_poly_act_deg7(ctx, [d_cts[i % 2] for i in range(n_ct)], level, k, rlk, ws=ws, merged=merged)
        ok = all(np.array_equal(hx.to_host(o), want[merged][i % 2]) for i, o in enumerate(outs))
        assert ok and untouched(buf), f"merged = {merged}"


@pytest.mark.parametrize("log_n,bits", [(13, 50), (12, 50), (11, 50), (13, 57)])
def test_rotations_stay_within_their_workspace(log_n, bits):
    """The scratch of unhoisted rotations is their key switches', plus a permuted copy of each polynomial only where no transform gathers it: five
    rotations with exactly the queried bytes, and in the size for one, give the oracle's residues and touch nothing around
    them.  Hoisted ones likewise in the least that is accepted: one decomposition and the inner products of the call."""
    p = make_params(log_n, 6, 2, 3, bits=bits)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(7300 + log_n + bits)
    level, n, offs = p.num_q - 1, orc.N, [3, -1, 7, 2, -9]
    L1, E, beta = level + 1, level + 1 + p.num_p, 3
    one = hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_KEYSWITCH, level)
    assert one == 8 * n * (L1 + beta * E + 2 * E + 2 * L1)
    copies = 0 if bits == 50 and log_n > 11 else 8 * n * L1
    for m in (1, 5, 8) + ((16,) if not copies else ()):
        assert hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_ROTATE, level, m) == m * (one + copies)
    ct = rand_ct(rng, p.moduli, level, n)
    d_ct = hx.from_host(ct)
    keys = [np.stack([np.stack([rand_poly(rng, p.moduli, n) for _ in range(2)]) for _ in range(p.dnum)]) for _ in offs]
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(k), hx.ckks_galois_element(ctx, r)) for k, r in zip(keys, offs)]
    want = orc.rotate_many(ct, level, offs, keys, False)
    least = 8 * n * (L1 + beta * E + 2 * len(offs) * (E + L1))
    for hoisted, nbytes in ((False, 5 * (one + copies)), (False, one + copies), (True, least)):
        buf = torch.full((nbytes // 8 + 128,), 0x5A5A5A5A, dtype=torch.int64, device="cuda")
        outs = hx.ckks_rotate_hoisted(ctx, d_ct, level, offs, dkeys, hoisted, ws=buf[64:-64])
        assert all(np.array_equal(hx.to_host(o), w) for o, w in zip(outs, want)), f"hoisted = {hoisted}, {nbytes} bytes"
        assert bool((buf[:64] == 0x5A5A5A5A).all()) and bool((buf[-64:] == 0x5A5A5A5A).all()), f"hoisted = {hoisted}, {nbytes} bytes"
    for hoisted, nbytes in ((False, one + copies - 256), (True, least - 256)):
        with pytest.raises(hx.CkksError) as e:
            hx.ckks_rotate_hoisted(ctx, d_ct, level, offs, dkeys, hoisted, ws=hx.empty(nbytes // 8))
        assert e.value.code == hx.binding.CKKS_ERR_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level,n_ct", [(13, 6, 2, 3, 5, 1), (13, 5, 5, 1, 4, 3), (14, 9, 3, 3, 6, 8), (13, 19, 2, 10, 18, 2),
                                                               (15, 7, 3, 3, 5, 1)])
def test_inner_products_go_on_into_the_inverse_pass(log_n, num_q, num_p, dnum, level, n_ct):
    """The sums of the limbs that the division behind drops leave the fused inner product with the first pass of their inverse
    transform done: special primes alone (product, unhoisted rotations) and with the level's own limb (merged activation),
    whose sum has no transformed digit where there is one digit; one item per workgroup and several; ten digits."""
    p = make_params(log_n, num_q, num_p, dnum)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(8000 + log_n * 10 + dnum)
    cts = [rand_ct(rng, p.moduli, level, orc.N) for _ in range(2)]
    d_cts = [hx.from_host(c) for c in cts]
    offs = [3, -1, 7][:1 + n_ct % 3]
    keys = [np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(dnum)]) for _ in range(1 + len(offs))]
    rlk = hx.ckks_key_load(ctx, hx.from_host(keys[0]), 0)
    got = hx.ckks_ctct_mul_relin(ctx, d_cts[0], d_cts[1], level, rlk)
    assert np.array_equal(hx.to_host(got), orc.ctct_mul_relin(*cts, keys[0], level))
    rot = [hx.ckks_key_load(ctx, hx.from_host(k), hx.ckks_galois_element(ctx, r)) for k, r in zip(keys[1:], offs)]
    outs = hx.ckks_rotate_hoisted(ctx, d_cts[0], level, offs, rot, False)
    for out, want in zip(outs, orc.rotate_many(cts[0], level, offs, keys[1:], False)):
        assert np.array_equal(hx.to_host(out), want)
    k = (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
    want = [orc.poly_activation_merged(c, level, k, keys[0]) for c in cts]
    outs = hx.he_poly_act_deg7(ctx, [d_cts[i % 2] for i in range(n_ct)], level, k, rlk, merged=True)
    for i, out in enumerate(outs):
        assert np.array_equal(hx.to_host(out), want[i % 2]), f"ciphertext {i}"


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level", [(12, 5, 1, 5, 4), (12, 12, 12, 1, 11), (12, 16, 14, 1, 15), (12, 25, 9, 3, 24), (13, 10, 10, 1, 9), (13, 11, 9, 2, 10), (13, 5, 1, 5, 4), (14, 9, 4, 3, 8), (14, 6, 6, 1, 5),
                                                          (15, 5, 1, 5, 4), (15, 5, 8, 2, 4), (15, 13, 5, 3, 12), (16, 5, 1, 5, 4), (17, 3, 2, 2, 2)])
def test_inverse_pass_inside_the_conversion(log_n, num_q, num_p, dnum, level):
    """The inverse transform's second pass inside the converting first pass and on its own: one source limb (rescales; digits of one limb,
    each with a modulus of its own), ragged digits, up to sixteen source limbs of the ring of 2^12 points, the most points a thread takes on the small rings (ten limbs of four, five of
    eight) and one more (six of eight: pass by pass), two to nine limbs through LDS with one group of targets (eight special primes and
    the level's limb in a merged division) and more, N = 2^17."""
    p = make_params(log_n, num_q, num_p, dnum)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(9000 + log_n * 10 + num_q)
    ct = rand_ct(rng, p.moduli, level, orc.N)
    d_ct = hx.from_host(ct)
    key = np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(dnum)])
    dkey = hx.ckks_key_load(ctx, hx.from_host(key), hx.ckks_galois_element(ctx, 3))
    for lv in {level, 1, level // 2 + 1}:
        c = np.ascontiguousarray(ct[:, :lv + 1])
        assert np.array_equal(hx.to_host(hx.ckks_rescale(ctx, hx.from_host(c), lv)), orc.rescale(c, lv)), f"rescale from level {lv}"
    for hoisted in (True, False):
        (got,) = hx.ckks_rotate_hoisted(ctx, d_ct, level, [3], [dkey], hoisted)
        assert np.array_equal(hx.to_host(got), orc.rotate_many(ct, level, [3], [key], hoisted)[0]), f"hoisted = {hoisted}"
    if level >= 4:
        k = (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
        (got,) = hx.he_poly_act_deg7(ctx, [d_ct], level, k, hx.ckks_key_load(ctx, hx.from_host(key), 0), merged=True)
        assert np.array_equal(hx.to_host(got), orc.poly_activation_merged(ct, level, k, key)), "activation"


def test_rescales_of_the_whole_ring_kernel():
    """N = 2^12: a rescale is one launch up to 256 limb-polys of results (a single output), pass by pass above (eight outputs of 17
    limbs); its input's last limb at the extremes."""
    p = make_params(12, 18, 6, 3)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(9500)
    level, q = 17, p.moduli
    ct = rand_ct(rng, q, level, orc.N)
    offs = conv_tap_offsets(4)
    keys = {o: np.stack([np.stack([rand_poly(rng, q, orc.N) for _ in range(2)]) for _ in range(p.dnum)]) for o in offs if o}
    masks = np.stack([rand_poly(rng, q[:level + 1], orc.N) for _ in range(9)])
    w = rng.integers(-2 ** 31, 2 ** 31, size=(9, 1, 9))
    want = orc.he_conv([ct], level, 4, keys, masks, w)
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(keys[o]), hx.ckks_galois_element(ctx, o)) if o else None for o in offs]
    outs = hx.he_conv_batched(ctx, 4, 4, 2, level, [hx.from_host(ct)], dkeys, hx.from_host(masks), hx.from_host(w_residues(w, q, level)), 9)
    for o in range(9):
        assert np.array_equal(hx.to_host(outs[o]), want[o]), f"output {o}"
    ct[:, level, :3] = [[0, q[level] - 1, q[level] // 2]] * 2
    for lv in (1, 7, level):
        c = np.ascontiguousarray(ct[:, :lv + 1])
        assert np.array_equal(hx.to_host(hx.ckks_rescale(ctx, hx.from_host(c), lv)), orc.rescale(c, lv))


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level", [(12, 6, 2, 3, 5), (12, 7, 1, 7, 6), (13, 24, 8, 3, 22)])
def test_more_than_eight_items_in_a_call(log_n, num_q, num_p, dnum, level):
    """Up to sixteen items share every launch: rotations (hoisted in launches of eight taps, unhoisted), activation of eleven and of five (the
    two middle products of a ciphertext in one batch), merge of eleven blocks, fully connected layer with eleven outputs, and convolutions
    from and to eleven channels; in the queried workspace and in the one that batches of eight need; seven digits; a ring where
    the activation alternates between two streams (convolutions that do: test_convolutions_on_two_streams)."""
    p = make_params(log_n, num_q, num_p, dnum)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(9700 + log_n + dnum)
    q, n = p.moduli, orc.N
    pt = lambda lv: rand_poly(rng, q[:lv + 1], n)
    keys, dkeys = {}, {}

    def key(r):
        if r % orc.n == 0:
            return None
        if r not in keys:
            keys[r] = np.stack([np.stack([rand_poly(rng, q, n) for _ in range(2)]) for _ in range(dnum)])
            dkeys[r] = hx.ckks_key_load(ctx, hx.from_host(keys[r]), hx.ckks_galois_element(ctx, r))
        return dkeys[r]

    same = lambda got, want: bool(np.array_equal(hx.to_host(got), want))
    cts = [rand_ct(rng, q, level, n) for _ in range(3)]
    d_cts = [hx.from_host(c) for c in cts]
    beta = lambda lv: -(-(lv + 1) // -(-num_q // dnum))
    ks = lambda lv, nd, nv: 8 * n * (nd * (lv + 1) + nd * beta(lv) * (lv + 1 + num_p) + nv * 2 * (2 * lv + 2 + num_p))  # a key switch's scratch
    offs = [1 + 3 * i for i in range(11)]
    dk = [key(r) for r in offs]
    want = orc.rotate_many(cts[0], level, offs, [keys[r] for r in offs], True)
    full = hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_ROTATE, level, 11)
    for hoisted in (True, False):
        for nbytes in (full, hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_ROTATE, level, 8)):
            outs = hx.ckks_rotate_hoisted(ctx, d_cts[0], level, offs, dk, hoisted, ws=hx.empty(nbytes // 8))
            assert all(same(o, w) for o, w in zip(outs, want)), f"rotations, hoisted = {hoisted}, {nbytes} bytes"
    rlk = np.stack([np.stack([rand_poly(rng, q, n) for _ in range(2)]) for _ in range(dnum)])
    d_rlk, k = hx.ckks_key_load(ctx, hx.from_host(rlk), 0), (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
    want = [orc.poly_activation_merged(c, level, k, rlk) for c in cts[:2]]
    for n_ct in (11, 5):
        full = hx.ckks_workspace_bytes(ctx, hx.CKKS_OP_POLY_ACT, level, n_ct)
        m = min(n_ct, 8)  # a batch without the pairs of products
        small = 8 * n * 2 * m * (level + 2 * (level - 1) + level - 2 + level + 1) + ks(level, m, m) + 8 * n * 2 * m * (1 + level) + 4096
        assert small < full
        for nbytes in (full, small):
            outs = hx.he_poly_act_deg7(ctx, [d_cts[i % 2] for i in range(n_ct)], level, k, d_rlk, ws=hx.empty(nbytes // 8), merged=True)
            assert all(same(o, want[i % 2]) for i, o in enumerate(outs)), f"activation of {n_ct}, {nbytes} bytes"
    if level > 8:
        return
    sts, mask = orc.n // 16, pt(level)
    got = hx.he_accumulator_merge(ctx, [d_cts[i % 3] for i in range(11)], level, sts, hx.from_host(mask), [key(-i * sts) for i in range(11)])
    assert same(got, orc.accumulator_merge([cts[i % 3] for i in range(11)], level, sts, mask, keys)), "merge"
    d_in, d_out, batch, base = 16, 11, 6, 3
    _, lo, hi = orc.fc_shifts(d_in, d_out, batch, base)
    ops = (np.stack([pt(level) for _ in range(d_out)]), pt(level - 1), np.stack([pt(level - 2) for _ in range(batch)]), pt(level - 3))
    fc_keys = ([key(1 << s) for s in range(4)], [key(-i) for i in range(d_out)], [key(r) for r in lo], [key(r) for r in hi])
    want = orc.fc_batched(cts[0], level, d_in, d_out, batch, base, *ops, keys)
    full = hx.he_fc_workspace_bytes(ctx, d_in, d_out, batch, level, base)
    for nbytes in (full, full - 8 * n * 3 * 2 * (2 * level + num_p)):  # room for the eight, not for the eleven
        got = hx.he_fc_batched(ctx, d_cts[0], level, d_in, d_out, batch, base, *[hx.from_host(o) for o in ops], *fc_keys, ws=hx.empty(nbytes // 8))
        assert same(got, want), f"fully connected layer, {nbytes} bytes"
    toffs = conv_tap_offsets(4)
    tkeys = [key(o) for o in toffs]
    for c_in, c_out in ((11, 2), (2, 11)):
        w = rng.integers(-2 ** 31, 2 ** 31, size=(c_out, c_in, 9))
        ins = [cts[i % 3] for i in range(c_in)]
        for al in (hx.HE_CONV_ALIGN_DIRECT, hx.HE_CONV_DEFERRED_MODDOWN, hx.HE_CONV_DEFERRED_MERGED):
            ext = al != hx.HE_CONV_ALIGN_DIRECT
            idx = orc.ext_moduli_idx(level) if ext else list(range(level + 1))
            masks = np.stack([rand_poly(rng, [q[t] for t in idx], n) for _ in range(9)])
            w_res = np.array([[[[int(w[o, i, t]) % q[m] for m in idx] for t in range(9)] for i in range(c_in)] for o in range(c_out)], dtype=np.uint64)
            want = orc.he_conv_deferred(ins, level, 4, keys, masks, w, merged=al == hx.HE_CONV_DEFERRED_MERGED) if ext else orc.he_conv(ins, level, 4, keys, masks, w)
            outs = hx.he_conv_batched(ctx, 4, 4, 2, level, [d_cts[i % 3] for i in range(c_in)], tkeys, hx.from_host(masks), hx.from_host(w_res), c_out, alignment=al)
            assert all(same(o, want[i]) for i, o in enumerate(outs)), f"convolution {c_in} -> {c_out}, schedule {al}"


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,c_in,c_out,limit", [(13, 3, 2, 2, 17, 2, 15), (15, 4, 2, 2, 9, 2, 17), (15, 4, 2, 2, 2, 17, 17),
                                                                         (16, 7, 2, 4, 1, 9, 19)])
def test_convolutions_on_two_streams(log_n, num_q, num_p, dnum, c_in, c_out, limit):
    """Deferred convolutions whose batches of input channels, or of output channels, alternate between the context's two streams: more than eight
    of either on rings above the size up to which they go together (2^17 coefficients of the extended basis, 2^15 from more than sixteen
    channels, 2^19 where the merged divisions alone come in batches and sixteen would hold them); with the overlap on, off and on
    again, and replayed from a graph."""
    p = make_params(log_n, num_q, num_p, dnum)
    assert (num_q + num_p) << log_n > 1 << limit
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(9900 + log_n + c_in)
    level, q, n = p.num_q - 1, p.moduli, orc.N
    toffs = conv_tap_offsets(4)
    keys = {o: np.stack([np.stack([rand_poly(rng, q, n) for _ in range(2)]) for _ in range(dnum)]) for o in toffs if o}
    dkeys = [hx.ckks_key_load(ctx, hx.from_host(keys[o]), hx.ckks_galois_element(ctx, o)) if o else None for o in toffs]
    cts = [rand_ct(rng, q, level, n) for _ in range(c_in)]
    d_in = [hx.from_host(c) for c in cts]
    idx = orc.ext_moduli_idx(level)
    masks = np.stack([rand_poly(rng, [q[t] for t in idx], n) for _ in range(9)])
    w = rng.integers(-2 ** 31, 2 ** 31, size=(c_out, c_in, 9))
    d_masks, d_w = hx.from_host(masks), hx.from_host(w_residues(w, [q[t] for t in idx], len(idx) - 1))
    for al in (hx.HE_CONV_DEFERRED_MERGED, hx.HE_CONV_DEFERRED_MODDOWN):
        want = orc.he_conv_deferred(cts, level, 4, keys, masks, w, merged=al == hx.HE_CONV_DEFERRED_MERGED)
        outs = [hx.empty(2, level, n) for _ in range(c_out)]
        ws = hx.empty(hx.he_conv_workspace_bytes(ctx, c_in, c_out, 4, 4, 2, level, al) // 8 + 1)
        st = torch.cuda.Stream()
        torch.cuda.synchronize()
        run = lambda: hx.he_conv_batched(ctx, 4, 4, 2, level, d_in, dkeys, d_masks, d_w, c_out, outs=outs, ws=ws, alignment=al, stream=st.cuda_stream)

        def check(what):
            st.synchronize()
            assert all(np.array_equal(hx.to_host(o), want[i]) for i, o in enumerate(outs)), f"{what}, schedule {al}"
            for o in outs:
                o.zero_()
            torch.cuda.synchronize()

        for on in (True, False, True):
            hx.ckks_ctx_set_overlap(ctx, on)
            run()
            check(f"overlap {on}")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            run()
        for _ in range(3):
            torch.randn(1 << 16, device="cuda").sum().item()  # eager work and a synchronisation between replays
            graph.replay()
            torch.cuda.synchronize()
            check("replay")
