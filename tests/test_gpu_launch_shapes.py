"""GPU parity at the sizes where the launch rules change: how many batch items a lo-pass workgroup takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2604_16834_amd as hx  # noqa: E402
from oracle import Oracle  # noqa: E402
from workloads import make_params  # noqa: E402
from gpu_common import rand_poly  # noqa: E402


@pytest.mark.parametrize("batch,bits", [(191, 50), (383, 50), (384, 50), (385, 57), (577, 50), (1537, 50)])
def test_ntt_items_per_workgroup(batch, bits):
    """Four slices at N = 2^12: one item per workgroup below 384 polynomials, two from there (the inverse pass' most), three at
    577 with a ragged last share, eight (the forward pass' most) with a workgroup of one at 1537."""
    p = make_params(12, 2, 1, 1, bits=bits)
    orc, ctx = Oracle(p), hx.Context(p)
    rng = np.random.default_rng(2000 + batch)
    idx = [2, 1]
    polys = np.stack([rand_poly(rng, [p.moduli[t] for t in idx], orc.N) for _ in range(batch)])
    d = hx.from_host(polys)
    hx.ckks_ntt_fwd(ctx, d, idx)
    assert np.array_equal(hx.to_host(d), orc.ntt_many(polys, idx))
    hx.ckks_ntt_inv(ctx, d, idx)
    assert np.array_equal(hx.to_host(d), polys)
