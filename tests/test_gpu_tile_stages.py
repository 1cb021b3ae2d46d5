"""bf16 sets on 64- and 128-tiles: symmetric outputs whose 64-tiles fit one round
run on these, other launches on 128-tiles with four LDS stages for at most 256 of
them, else two. The products are formed in the same order, so
a matrix on its own and among many equal ones gets the same value and gradient
bit for bit; and both agree with the oracle."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from oracle.pe_schedule import default_table  # noqa: E402
from oracle.slorr import fwd_bwd  # noqa: E402

pytestmark = pytest.mark.gpu


# one k-slab pair (128); fewer and more slabs than stages; ragged edges; a single row
@pytest.mark.parametrize("shape", [(100, 128), (128, 100), (200, 300), (384, 640), (650, 1300), (1, 257)])
@pytest.mark.parametrize("iters", [1, 3])
def test_four_and_two_stages_agree(shape, iters):
    """Against the oracle: the 2e-2 bar of bf16 sets."""
    import torch
    from paper_2607_08754_amd.slorr import Plan

    rng = np.random.default_rng(shape[0] * 7 + shape[1] + iters)
    w = torch.tensor(rng.standard_normal(shape), dtype=torch.float32, device="cuda").mul_(0.02).bfloat16()

    def run(n):
        weights = [w.clone() for _ in range(n)]
        grads = [torch.zeros(shape, device="cuda") for _ in range(n)]
        plan = Plan([shape] * n, dtype="bf16", device="cuda", kind="nuclear", iters=iters)
        vals = plan(weights, grads)
        return vals[:n].cpu().numpy(), [g.cpu().numpy() for g in grads]

    one_v, one_g = run(1)
    many_v, many_g = run(300)
    assert np.all(many_v == one_v[0])
    for g in many_g:
        assert np.array_equal(g, one_g[0])

    ref = fwd_bwd(w.double().cpu().numpy(), "nuclear", default_table(iters))
    assert abs(one_v[0] - ref.value) <= 2e-2 * abs(ref.value)
    assert np.linalg.norm(one_g[0] - ref.grad) <= 2e-2 * np.linalg.norm(ref.grad)
