"""GPU parity where a call takes another route through the kernels for its size or its operands."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2604_16834_amd as hx  # noqa: E402
from oracle import Oracle  # noqa: E402
from workloads import make_params  # noqa: E402


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
