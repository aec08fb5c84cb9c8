"""The algorithmic bytes and butterflies that ckks_prof_end reports for the transforms' last forward pass (class ntt_fwd_lo), which takes inner products
and the ends of divisions with it: every launch is charged with the positions that it covers, counted here limb by limb."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2604_16834_amd as hx  # noqa: E402
from workloads import make_params  # noqa: E402
from test_gpu_call_paths import uniform  # noqa: E402


class Shape:
    """A context at a level: L1 limbs that stay, k that a division drops, E positions in beta digits; keys and ciphertexts to call it with."""

    def __init__(self, log_n, num_q, num_p, dnum, seed):
        self.ctx = hx.Context(make_params(log_n, num_q, num_p, dnum))
        self.log_n, self.dnum, self.level, self.L1, self.k = log_n, dnum, num_q - 1, num_q, num_p
        self.E, self.beta = num_q + num_p, -(-num_q // -(-num_q // dnum))
        self.residues, _ = uniform(self.ctx, make_params(log_n, num_q, num_p, dnum), seed)

    def ct(self):
        return self.residues(2, limbs=list(range(self.L1)))

    def key(self, offset=None):
        t = self.residues(self.dnum, 2, limbs=list(range(self.ctx.M)))
        return hx.ckks_key_load(self.ctx, t, 0 if offset is None else hx.ckks_galois_element(self.ctx, offset))

    def check(self, call, rows, transforms):
        """rows: limb-polys read and written by the class, transforms: limb-polys that go through 2^11-point passes."""
        hx.ckks_ctx_set_overlap(self.ctx, False)
        hx.ckks_prof_begin(self.ctx, ["ntt_fwd_lo"])
        call()
        got = hx.ckks_prof_end(self.ctx)
        assert got["dropped"] == 0
        assert got["ntt_fwd_lo"]["bytes"] == 8 * self.ctx.N * rows
        assert got["ntt_fwd_lo"]["ops"] == self.ctx.N // 2 * 11 * transforms


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,n", [(13, 14, 5, 3, 8), (15, 8, 3, 3, 8)])
def test_hoisted_rotations(log_n, num_q, num_p, dnum, n):
    """All positions in one launch, whose sums a division then reads (448 slices), and in two launches around the division (1024)."""
    s = Shape(log_n, num_q, num_p, dnum, 1)
    offs = list(range(1, n + 1))
    ct, keys = s.ct(), [s.key(o) for o in offs]
    own = s.beta * s.E - s.L1  # the digits' last pass, in and out
    # digits with their own limbs and c0 once for all, keys and sums per rotation
    rows = 2 * own + s.beta * s.E + s.L1 + n * 2 * s.beta * s.E
    if s.L1 * n << (log_n - 11) < 900:
        rows += n * 2 * s.E + 3 * n * 2 * s.L1  # converted part, sums, results
    else:
        rows += n * 2 * s.k + 2 * n * 2 * s.L1  # the dropped limbs' sums; converted part, results
    s.check(lambda: hx.ckks_rotate_hoisted(s.ctx, ct, s.level, offs, keys, True), rows, own + n * 2 * s.E)


@pytest.mark.parametrize("log_n,num_q,num_p,dnum,n", [(13, 6, 3, 2, 3), (14, 10, 4, 3, 10)])
def test_rotations_of_one_ciphertext(log_n, num_q, num_p, dnum, n):
    """Each with its own digits, 72 and 800 slices."""
    s = Shape(log_n, num_q, num_p, dnum, 2)
    offs = list(range(1, n + 1))
    ct, keys = s.ct(), [s.key(o) for o in offs]
    own = s.beta * s.E - s.L1
    rows = n * own + 2 * s.L1 + n * 2 * s.beta * s.E + n * 2 * s.k + 4 * n * s.L1 + (2 * n * s.L1 if s.L1 * n << (log_n - 11) < 768 else 0)
    rows += 2 * n * s.L1 if s.L1 * n << (log_n - 11) < 768 else 0
    s.check(lambda: hx.ckks_rotate_hoisted(s.ctx, ct, s.level, offs, keys, False), rows, n * (own + 2 * s.E))


@pytest.mark.parametrize("log_n,num_q,num_p,dnum", [(13, 6, 3, 2), (16, 24, 8, 3)])
def test_product(log_n, num_q, num_p, dnum):
    s = Shape(log_n, num_q, num_p, dnum, 3)
    a, b, rlk = s.ct(), s.ct(), s.key()
    own = s.beta * s.E - s.L1
    rows = own + 4 * s.L1 + 2 * s.beta * s.E + 2 * s.k + 4 * s.L1 + (4 * s.L1 if s.L1 << (log_n - 11) < 768 else 0)
    s.check(lambda: hx.ckks_ctct_mul_relin(s.ctx, a, b, s.level, rlk), rows, own + 2 * s.E)


def test_merge():
    """Three rotations whose masked products are formed where they are read, three partial sums, one division, a rescale."""
    s = Shape(13, 10, 4, 3, 4)
    sts = s.ctx.N // 8
    cts, mask, keys = [s.ct() for _ in range(4)], s.residues(limbs=list(range(s.L1))), [None] + [s.key(-i * sts) for i in range(1, 4)]
    own = s.beta * s.E - s.L1
    rows = 3 * own + 3 * 2 * s.L1 + s.L1 + 3 * 2 * s.beta * s.E + 3 * 2 * s.E  # inner products
    rows += 2 * s.L1 + 3 * 2 * s.L1 + 2 * s.L1 + s.L1 + 2 * s.L1  # converted part, partial sums, the block that stays, its mask; the sum
    rows += 3 * 2 * s.level  # rescale: converted limb, others, results
    s.check(lambda: hx.he_accumulator_merge(s.ctx, cts, s.level, sts, mask, keys), rows, 3 * own + 3 * 2 * s.k + 2 * s.L1 + 2 * s.level)
