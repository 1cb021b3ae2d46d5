"""Update launches on 256-tiles with edge tiles (padded dims that are no
multiples of 256), against the same iteration in float64."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from oracle.pe_schedule import default_table  # noqa: E402

pytestmark = pytest.mark.gpu


# half tiles at the right edge, at the lower edge, at both; tall matrices;
# a set of mixed shapes, whole tiles among them
@pytest.mark.parametrize("shapes", [[(1280, 3456)] * 8, [(1152, 2048)] * 14, [(3456, 1152)] * 9,
                                    [(1280, 1280), (3456, 1280), (1280, 3400), (1024, 2048)] * 4])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_edge_tiles(shapes, dtype):
    """Gradient and value at the size of the iterate's rounding (split: 2e-5
    and 1e-6; fp16: the 2e-2 bar, a tenth of it for the values)."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(19)
    W = [(torch.randn(s, generator=gen, device="cuda:0") * 0.02).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
         for s in shapes]
    G = [torch.empty(s, device="cuda:0") for s in shapes]
    plan = Plan(shapes, dtype=dtype, iters=6)
    assert any(op == "update" and edge == 256 for op, _, edge in plan.launches())
    vals = plan(W, G).double()
    gtol, vtol = (2e-2, 2e-3) if dtype == "bf16" else (2e-5, 1e-6)
    for i, (w, s) in enumerate(zip(W, shapes)):
        w = w.double()
        y = w if s[0] <= s[1] else w.t().contiguous()
        f = y.norm()
        x = y / f
        for a, b, c in default_table(6):
            sq = x @ x.t()
            x = a * x + (b * sq + c * (sq @ sq)) @ x
        nh = (y * x).sum()
        g = 2 * nh / f ** 2 * x - 2 * nh ** 2 / f ** 4 * y
        g = g if s[0] <= s[1] else g.t()
        assert abs(vals[i] - (nh / f) ** 2) <= vtol * (nh / f) ** 2, i
        assert (G[i] - g).norm() <= gtol * g.norm(), i
