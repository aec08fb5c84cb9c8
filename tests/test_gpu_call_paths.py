"""GPU parity where a call takes another route through the kernels for its size or its operands."""
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


@pytest.mark.parametrize("batch", [141, 143])
def test_large_ntt_batches_in_parts(batch):
    """24 limbs at N = 2^14: 443.5 MB go through at once, 449.8 MB in parts of 72 and 71 polynomials.  The polynomials at the ends and at the
    cut against the oracle, all of them back through the inverse."""
    p = make_params(14, 24, 0, 0)
    orc, ctx = Oracle(p), hx.Context(p)
    idx = list(range(24))
    gen = torch.Generator(device="cuda").manual_seed(batch)
    q = torch.tensor(p.moduli, dtype=torch.int64, device="cuda")
    d = torch.randint(0, (1 << 63) - 1, (batch, 24, orc.N), generator=gen, device="cuda").remainder_(q.unsqueeze(-1))
    first = d.clone()
    hx.ckks_ntt_fwd(ctx, d, idx)
    for b in (0, 71, 72, batch - 1):
        assert np.array_equal(hx.to_host(d[b]), orc.ntt_many(hx.to_host(first[b])[None], idx)[0]), b
    hx.ckks_ntt_inv(ctx, d, idx)
    assert torch.equal(d, first)


def deferred_conv(ctx, p, level, width, cts, keys, masks, w, merged, ws=None):
    """cts, masks: on the device; keys by offset, None where nothing is rotated; w [c_out][c_in][9] integers."""
    ext = [p.moduli[t] for t in list(range(level + 1)) + list(range(p.num_q, p.num_q + p.num_p))]
    offs = conv_tap_offsets(width)
    dkeys = [hx.ckks_key_load(ctx, keys[o], hx.ckks_galois_element(ctx, o)) if o in keys else None for o in offs]
    outs = hx.he_conv_batched(ctx, 1, width, 1, level, cts, dkeys, masks, hx.from_host(w_residues(w, ext, len(ext) - 1)), w.shape[0],
                              alignment=hx.HE_CONV_DEFERRED_MERGED if merged else hx.HE_CONV_DEFERRED_MODDOWN, ws=ws)
    return [hx.to_host(o) for o in outs]


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level,c_in,c_out,merged",
                         [(12, 4, 2, 2, 3, 1, 1, True), (12, 5, 2, 3, 4, 3, 8, True), (12, 4, 1, 4, 3, 2, 5, False), (6, 3, 2, 2, 2, 3, 2, True),
                          (13, 3, 3, 1, 2, 5, 3, True)])
def test_inner_products_and_sum_in_one_kernel(log_n, num_q, num_p, dnum, level, c_in, c_out, merged):
    """One to four digits, one to four outputs per thread and two groups of outputs (5, 8), channels in ones, twos and threes with a ragged
    last pair, a ring of one workgroup per limb; uniform operands, weights of both signs up to 2^48."""
    p = make_params(log_n, num_q, num_p, dnum)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(100 * c_in + c_out)
    ext = [p.moduli[t] for t in orc.ext_moduli_idx(level)]
    cts = [rand_ct(rng, p.moduli, level, orc.N) for _ in range(c_in)]
    keys = {o: np.stack([np.stack([rand_poly(rng, p.moduli, orc.N) for _ in range(2)]) for _ in range(dnum)]) for o in conv_tap_offsets(4) if o}
    masks = np.stack([rand_poly(rng, ext, orc.N) for _ in range(9)])
    w = rng.integers(-2 ** 48, 2 ** 48, size=(c_out, c_in, 9))
    want = orc.he_conv_deferred(cts, level, 4, keys, masks, w, merged=merged)
    got = deferred_conv(ctx, p, level, 4, [hx.from_host(c) for c in cts], {o: hx.from_host(k) for o, k in keys.items()}, hx.from_host(masks), w, merged)
    for o in range(c_out):
        assert np.array_equal(got[o], want[o]), f"output {o}"


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level,width,c_in,c_out",
                         [(12, 5, 2, 3, 4, 2048, 2, 2), (13, 6, 2, 4, 5, 8, 19, 4), (13, 9, 3, 3, 6, 8, 33, 1), (14, 20, 5, 4, 17, 16, 9, 2),
                          (15, 7, 2, 4, 6, 8, 16, 3), (16, 12, 8, 2, 11, 8, 9, 4), (16, 12, 12, 1, 11, 8, 17, 1), (16, 6, 2, 3, 5, 8, 6, 4),
                          (12, 3, 3, 1, 2, 8, 12, 4)])
@pytest.mark.parametrize("low", [False, True])
def test_inner_products_and_sum_equal_stored_copies(log_n, num_q, num_p, dnum, level, width, c_in, c_out, low):
    """Against the same layer with enough outputs for the stored copies, whose first outputs are the same: three taps without a rotation (rows as
    long as the slots), more channels than a launch takes (the sums go on from the last one's), one wavefront for all taps of several
    outputs and three; every operand at q - 1 (low: at 0 and 1 in turn) beside uniform ones."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx = hx.Context(p)
    gen = torch.Generator(device="cuda").manual_seed(c_in)
    live = list(range(level + 1))
    q = torch.tensor(p.moduli, dtype=torch.int64, device="cuda")

    def residues(*lead, limbs):
        r = torch.randint(0, (1 << 63) - 1, (*lead, len(limbs), ctx.N), generator=gen, device="cuda").remainder_(q[limbs].unsqueeze(-1))
        edge = (torch.arange(1024, device="cuda") & 1).expand(len(limbs), 1024) if low else (q[limbs] - 1).unsqueeze(-1).expand(len(limbs), 1024)
        r[..., 512:1536] = edge
        return r
    cts = [residues(2, limbs=live) for _ in range(c_in)]
    keys = {o: residues(dnum, 2, limbs=list(range(ctx.M))) for o in conv_tap_offsets(width) if o % (ctx.N // 2)}
    masks = residues(9, limbs=live + list(range(num_q, ctx.M)))
    w = np.random.default_rng(c_out).integers(-2 ** 31, 2 ** 31, size=(9, c_in, 9))
    few = deferred_conv(ctx, p, level, width, cts, keys, masks, w[:c_out], True)
    many = deferred_conv(ctx, p, level, width, cts, keys, masks, w, True)
    for o in range(c_out):
        assert np.array_equal(few[o], many[o]), f"output {o}"


def uniform(ctx, p, seed):
    """A source of [*lead][limbs][N] residues on the device; the first kilobyte of words is q - 1, the next 0 and 1 in turn."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = torch.tensor(p.moduli, dtype=torch.int64, device="cuda")

    def residues(*lead, limbs):
        r = torch.randint(0, (1 << 63) - 1, (*lead, len(limbs), ctx.N), generator=gen, device="cuda").remainder_(q[limbs].unsqueeze(-1))
        r[..., :128] = (q[limbs] - 1).unsqueeze(-1)
        r[..., 128:256] = torch.arange(128, device="cuda") & 1
        return r
    return residues, q


def guarded(nbytes):
    """A workspace of exactly so many bytes and the buffer around it."""
    buf = torch.full((nbytes // 8 + 128,), 0x5A5A5A5A, dtype=torch.int64, device="cuda")
    return buf, buf[64:-64]


def untouched(buf):
    return bool((buf[:64] == 0x5A5A5A5A).all()) and bool((buf[-64:] == 0x5A5A5A5A).all())


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,c_in,c_out,stored", [(12, 5, 2, 3, 20, 8, False), (13, 6, 2, 4, 19, 4, False), (15, 7, 2, 4, 17, 1, False), (13, 6, 2, 4, 19, 9, True)])
def test_deferred_convolutions_stay_within_their_workspace(log_n, num_q, num_p, dnum, c_in, c_out, stored):
    """With few outputs the queried workspace holds no aligned copies (nine per channel on the extended basis).  Exactly the queried bytes give the residues of
    a larger workspace and touch nothing around them."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx, level = hx.Context(p), num_q - 1
    residues, _ = uniform(ctx, p, log_n + c_out)
    live = list(range(level + 1))
    cts, masks = [residues(2, limbs=live) for _ in range(c_in)], residues(9, limbs=live + list(range(num_q, ctx.M)))
    keys = {o: residues(dnum, 2, limbs=list(range(ctx.M))) for o in conv_tap_offsets(4) if o}
    w = np.random.default_rng(c_in).integers(-2 ** 31, 2 ** 31, size=(c_out, c_in, 9))
    for merged in (True, False):
        nbytes = hx.he_conv_workspace_bytes(ctx, c_in, c_out, 1, 4, 1, level, hx.HE_CONV_DEFERRED_MERGED if merged else hx.HE_CONV_DEFERRED_MODDOWN)
        assert (nbytes >= c_in * 9 * 2 * (num_q + num_p) * ctx.N * 8) == stored
        want = deferred_conv(ctx, p, level, 4, cts, keys, masks, w, merged, hx.empty(nbytes // 4))
        buf, ws = guarded(nbytes)
        got = deferred_conv(ctx, p, level, 4, cts, keys, masks, w, merged, ws)
        assert untouched(buf)
        for o in range(c_out):
            assert np.array_equal(got[o], want[o]), f"output {o}"


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level,g,shared", [(12, 4, 1, 4, 3, 16, False), (12, 24, 8, 3, 20, 16, True), (12, 14, 14, 1, 13, 2, True), (13, 10, 5, 2, 9, 5, True),
                                                                   (14, 9, 9, 1, 7, 3, True), (14, 8, 2, 4, 3, 16, True), (15, 20, 7, 3, 18, 4, True), (16, 12, 4, 4, 11, 2, True),
                                                                   (16, 3, 3, 1, 2, 9, True), (16, 6, 3, 2, 5, 9, True), (16, 8, 4, 2, 7, 16, True), (17, 3, 2, 2, 2, 3, True)])
def test_merge_equals_its_steps(log_n, num_q, num_p, dnum, level, g, shared):
    """Products, rotations, sum and rescale one by one, on both sides of the line from which the rotations share a division: one item per partial sum, two,
    three and four with a ragged last one (the cases at 2^16 of 9 and 16 blocks), sums of up to fifteen, one to fourteen special primes, rings of two to 64 rows."""
    assert ((level + 1 + num_p) << log_n >= 3 << 15) == shared  # sums_together
    p = make_params(log_n, num_q, num_p, dnum)
    ctx = hx.Context(p)
    residues, q = uniform(ctx, p, 31 * g + log_n)
    live = list(range(level + 1))
    sts = ctx.N // 2 // g
    cts, mask = [residues(2, limbs=live) for _ in range(g)], residues(limbs=live)
    keys = [None] + [hx.ckks_key_load(ctx, residues(dnum, 2, limbs=list(range(ctx.M))), hx.ckks_galois_element(ctx, -i * sts)) for i in range(1, g)]
    got = hx.he_accumulator_merge(ctx, cts, level, sts, mask, keys)
    total = torch.zeros_like(cts[0])
    for i in range(g):
        t = hx.ckks_ptct_mac(ctx, [mask], [cts[i]], level)
        if i:
            t = hx.ckks_rotate_hoisted(ctx, t, level, [-i * sts], [keys[i]], False)[0]
        total = (total + t).remainder_(q[live].unsqueeze(-1))
    assert torch.equal(got, hx.ckks_rescale(ctx, total, level))


def test_merge_in_a_smaller_workspace():
    """Fifteen rotations that share a division, in the queried workspace (all at once) and in that of nine blocks (eight at a time): the second batch adds to
    the sum of the first, in place."""
    p = make_params(12, 24, 8, 3)
    ctx, level, g = hx.Context(p), 20, 16
    residues, _ = uniform(ctx, p, 77)
    live, sts = list(range(level + 1)), ctx.N // 2 // g
    cts, mask = [residues(2, limbs=live) for _ in range(g)], residues(limbs=live)
    keys = [None] + [hx.ckks_key_load(ctx, residues(3, 2, limbs=list(range(ctx.M))), hx.ckks_galois_element(ctx, -i * sts)) for i in range(1, g)]
    results = []
    for blocks in (g, 9):
        buf, ws = guarded(hx.he_accumulator_workspace_bytes(ctx, level, blocks))
        results.append(hx.he_accumulator_merge(ctx, cts, level, sts, mask, keys, ws=ws))
        assert untouched(buf)
    assert hx.he_accumulator_workspace_bytes(ctx, level, 9) < hx.he_accumulator_workspace_bytes(ctx, level, g)
    assert torch.equal(results[0], results[1])


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,c_in,c_out", [(12, 5, 2, 3, 18, 8), (15, 6, 2, 3, 3, 2)])
def test_few_outputs_in_a_captured_graph(log_n, num_q, num_p, dnum, c_in, c_out):
    """The one-kernel convolution captured and replayed between eager work, with other inputs at the last replay, against the eager call."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx, level = hx.Context(p), num_q - 1
    residues, _ = uniform(ctx, p, c_in)
    live, ext = list(range(level + 1)), list(range(num_q)) + list(range(num_q, ctx.M))
    cts, masks = [residues(2, limbs=live) for _ in range(c_in)], residues(9, limbs=ext)
    keys = [hx.ckks_key_load(ctx, residues(dnum, 2, limbs=list(range(ctx.M))), hx.ckks_galois_element(ctx, o)) if o else None for o in conv_tap_offsets(4)]
    w = hx.from_host(w_residues(np.random.default_rng(c_in).integers(-2 ** 31, 2 ** 31, size=(c_out, c_in, 9)), [p.moduli[t] for t in ext], len(ext) - 1))
    ws = hx.empty(hx.he_conv_workspace_bytes(ctx, c_in, c_out, 1, 4, 1, level, hx.HE_CONV_DEFERRED_MERGED) // 8 + 1)
    outs = [hx.empty(2, level, ctx.N) for _ in range(c_out)]
    st = torch.cuda.Stream()

    def run(to, stream):
        hx.he_conv_batched(ctx, 1, 4, 1, level, cts, keys, masks, w, c_out, outs=to, ws=ws, alignment=hx.HE_CONV_DEFERRED_MERGED, stream=stream)

    def eager():
        to = [hx.empty(2, level, ctx.N) for _ in range(c_out)]
        run(to, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return to

    want = eager()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        run(outs, st.cuda_stream)
    for replay in range(3):
        if replay == 2:
            for c in cts:
                c.copy_(residues(2, limbs=live))
            want = eager()
        for o in outs:
            o.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, v) for o, v in zip(outs, want)), replay


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,lo,hi", [(13, 5, 13, 3, [0, 5], [0, 7, 9]), (15, 5, 2, 3, [1], list(range(3, 40, 2))), (16, 5, 4, 3, [0, 3], [0, 0, 4, 0]),
                                                          (15, 5, 2, 3, [2], [0]), (15, 5, 2, 3, [2], [0] * 17 + [5, 6]), (12, 10, 1, 10, [0, 3, 4], [1, 2]), (13, 8, 1, 8, [0, 3], [1, 2])])
def test_layout_of_one_ciphertext_equals_that_of_two(log_n, num_q, num_p, dnum, lo, hi):
    """One ciphertext's second rotations are added up in the division; two, which share their keys, take them one by one.  With more blocks than a
    launch takes, several blocks that stay where they are, and nothing else; nine digits read through two first rotations, seven through one."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx = hx.Context(p)
    level = num_q - 2
    residues, _ = uniform(ctx, p, log_n + len(hi))
    live = list(range(level + 1))
    cts, keys = [residues(2, limbs=live) for _ in range(2)], {}
    for o in set(lo + hi) - {0}:
        keys[o] = hx.ckks_key_load(ctx, residues(dnum, 2, limbs=list(range(ctx.M))), hx.ckks_galois_element(ctx, o))
    masks = [[residues(limbs=live) for _ in lo] for _ in hi]
    run = lambda c: hx.he_relayout_two_rotations(ctx, c, level, lo, [keys.get(o) for o in lo], hi, [keys.get(o) for o in hi], masks)
    two = run(cts)
    for i in range(2):
        assert torch.equal(run(cts[i:i + 1])[0], two[i]), i


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,n_ct,stored", [(15, 5, 2, 3, 1, False), (16, 5, 4, 3, 1, False), (15, 5, 2, 3, 2, True), (12, 5, 2, 3, 1, True)])
def test_layouts_stay_within_their_workspace(log_n, num_q, num_p, dnum, n_ct, stored):
    """The queried workspace holds the second rotations' results only where they are stored: 2^12 points are below the line of shared divisions.  Exactly the
    queried bytes give the residues of a larger workspace and touch nothing around them."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx, level, lo, hi = hx.Context(p), num_q - 2, [0, 3], [0, 7, 9]
    nbytes = [hx.he_relayout_workspace_bytes(ctx, level, n_ct, len(lo), n) for n in (len(hi), len(hi) + 1)]
    per_block = [8 * n_ct * 2 * limbs * ctx.N for limbs in (level + 1, level, level)]  # a masked sum, rescaled, rotated
    assert nbytes[1] - nbytes[0] == sum(per_block if stored else per_block[:2])
    residues, _ = uniform(ctx, p, log_n)
    live = list(range(level + 1))
    cts = [residues(2, limbs=live) for _ in range(n_ct)]
    keys = {o: hx.ckks_key_load(ctx, residues(dnum, 2, limbs=list(range(ctx.M))), hx.ckks_galois_element(ctx, o)) for o in set(lo + hi) - {0}}
    masks = [[residues(limbs=live) for _ in lo] for _ in hi]
    buf, ws = guarded(nbytes[0])
    want, got = [hx.he_relayout_two_rotations(ctx, cts, level, lo, [keys.get(o) for o in lo], hi, [keys.get(o) for o in hi], masks, ws=w) for w in (hx.empty(nbytes[0] // 4), ws)]
    assert untouched(buf)
    for i in range(n_ct):
        assert torch.equal(got[i], want[i]), i


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level,n", [(13, 13, 5, 3, 12, 15), (14, 9, 3, 3, 8, 16), (15, 4, 4, 1, 3, 13), (15, 12, 3, 4, 9, 5), (17, 4, 2, 2, 3, 4)])
def test_rotations_together_equal_single_ones(log_n, num_q, num_p, dnum, level, n):
    """Enough unhoisted rotations for the inner products to wait for the division, against one at a time; no digit to transform, ragged last digits."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx = hx.Context(p)
    residues, _ = uniform(ctx, p, log_n)
    ct = residues(2, limbs=list(range(level + 1)))
    offs = [1 + 37 * i for i in range(n)]
    keys = [hx.ckks_key_load(ctx, residues(dnum, 2, limbs=list(range(ctx.M))), hx.ckks_galois_element(ctx, o)) for o in offs]
    got = hx.ckks_rotate_hoisted(ctx, ct, level, offs, keys, False)
    for i, o in enumerate(offs):
        assert torch.equal(got[i], hx.ckks_rotate_hoisted(ctx, ct, level, [o], [keys[i]], False)[0]), i


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level", [(13, 16, 6, 3, 15), (14, 14, 5, 3, 13), (15, 8, 8, 1, 7), (16, 7, 2, 4, 6)])
def test_activations_together_equal_single_ones(log_n, num_q, num_p, dnum, level):
    """Products with and without a linear addend whose inner products wait for the division (sixteen), against one ciphertext at a time."""
    p = make_params(log_n, num_q, num_p, dnum)
    ctx = hx.Context(p)
    residues, _ = uniform(ctx, p, log_n)
    cts = [residues(2, limbs=list(range(level + 1))) for _ in range(16)]
    rlk = hx.ckks_key_load(ctx, residues(dnum, 2, limbs=list(range(ctx.M))), 0)
    k = (3 << 40, -(5 << 40), 7 << 40, -(9 << 40))
    got = hx.he_poly_act_deg7(ctx, cts, level, k, rlk, merged=True)
    for i, c in enumerate(cts):
        assert torch.equal(got[i], hx.he_poly_act_deg7(ctx, [c], level, k, rlk, merged=True)[0]), i


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,level,n", [(12, 4, 1, 4, 3, 3), (12, 13, 13, 1, 12, 2), (13, 8, 4, 2, 7, 17), (14, 7, 3, 3, 5, 9), (15, 4, 2, 2, 3, 2), (16, 3, 3, 1, 1, 1),
                                                            (13, 15, 5, 3, 14, 16), (16, 4, 2, 2, 3, 8), (12, 30, 8, 4, 29, 16)])
def test_hoisted_rotations_of_every_row_count(log_n, num_q, num_p, dnum, level, n):
    """One set of digits read through each rotation, against the oracle: one to four digits, several batches, rings of two to 32
    rows, and enough of them for the inner products to wait for the division (the last three; on 2^12 points that takes sixteen of 29 limbs and more)."""
    p = make_params(log_n, num_q, num_p, dnum)
    orc, ctx = Oracle(p), hx.Context(p)
    residues, _ = uniform(ctx, p, n)
    ct = residues(2, limbs=list(range(level + 1)))
    offs = [1 + 61 * i * i for i in range(n)]
    raw = [residues(dnum, 2, limbs=list(range(ctx.M))) for _ in offs]
    got = hx.ckks_rotate_hoisted(ctx, ct, level, offs, [hx.ckks_key_load(ctx, k, hx.ckks_galois_element(ctx, o)) for k, o in zip(raw, offs)], True)
    host = hx.to_host(ct)
    digits = orc.modup(host[1], level)
    for i, o in enumerate(offs):
        assert np.array_equal(hx.to_host(got[i]), orc.rotate(host, level, o, hx.to_host(raw[i]), True, digits)), i
