"""Steps 1 and 2 formed on the Gram matrix (the default table of 6 and more
steps) against the same table given explicitly, which runs step by step, and
against the iteration in float64."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from oracle.pe_schedule import default_table  # noqa: E402

pytestmark = pytest.mark.gpu


def exact(w, kind, table):
    y = w if w.shape[0] <= w.shape[1] else w.t().contiguous()
    f = y.norm()
    x = y / f
    for a, b, c in table:
        sq = x @ x.t()
        x = a * x + (b * sq + c * (sq @ sq)) @ x
    n = (y * x).sum()
    if kind == "nuclear":
        v, g = n, x
    else:
        v, g = (n / f) ** 2, 2 * n / f ** 2 * x - 2 * n ** 2 / f ** 4 * y
    return v, (g if w.shape[0] <= w.shape[1] else g.t())


# one tile; several with edges, tall ones; split-K Gram; more tiles than CUs;
# 256-tiles with two per CU, whole and with edges; every step count parity
@pytest.mark.parametrize("shapes,iters", [
    ([(100, 600)] * 3, 6), ([(300, 2100), (2300, 130), (1, 700), (257, 2500)], 6), ([(100, 5000), (4200, 128)], 7),
    ([(384, 1000)] * 50, 8), ([(512, 2048)] * 64, 6), ([(2000, 600), (640, 2300)] * 24, 6)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind", ["hoyer", "nuclear"])
def test_chained_steps(shapes, iters, dtype, kind):
    """Each way is off by its roundings (bf16 sets: 2e-2, values 2e-3; fp32:
    5e-5, 1e-6); chained by no more than step by step (over a set; 15 % for the
    chance of one draw of roundings)."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(23)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    W = [(torch.randn(s, generator=gen, device="cuda:0") * 0.02).to(dt) for s in shapes]
    table = default_table(iters)
    got = []
    for coeffs in (None, table):
        G = [torch.full(s, float("nan"), device="cuda:0") for s in shapes]
        vals = Plan(shapes, dtype=dtype, kind=kind, iters=iters, coeffs=coeffs)(W, G)
        got.append((vals.double(), G))
    gtol, vtol = (2e-2, 2e-3) if dtype == "bf16" else (5e-5, 1e-6)
    err = [0.0, 0.0]
    size = 0.0
    for i, w in enumerate(W):
        v, g = exact(w.double(), kind, table)
        scale = g.norm() if min(w.shape) > 1 or kind == "nuclear" else 2 * v / w.double().norm()   # one row: g = 0
        size += float(scale) ** 2
        for q, (vals, G) in enumerate(got):
            d = (G[i].double() - g).norm()
            assert d <= gtol * scale, (q, i)
            assert abs(vals[i] - v) <= vtol * v, (q, i)
            err[q] += float(d) ** 2
    err = [(e / size) ** 0.5 for e in err]
    print(f"chained {err[0]:.3e} step by step {err[1]:.3e}", flush=True)
    assert err[0] <= 1.15 * err[1]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind", ["hoyer", "nuclear"])
def test_chained_special_values(dtype, kind):
    """A zero matrix, a NaN and an infinity among others stay their own (the
    nuclear gradient does not read W: its NaN comes through P)."""
    import torch
    from paper_2607_08754_amd import Plan
    shapes = [(200, 2000)] * 4
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    W = [(torch.randn(s, generator=gen, device="cuda:0") * 0.02).to(dt) for s in shapes]
    W[1].zero_()
    W[2][7, 11] = float("nan")
    W[3][0, 0] = float("inf")
    alone = torch.full(shapes[0], float("nan"), device="cuda:0")
    v0 = Plan(shapes[:1], dtype=dtype, kind=kind)(W[:1], [alone])
    G = [torch.full(s, float("nan"), device="cuda:0") for s in shapes]
    vals = Plan(shapes, dtype=dtype, kind=kind)(W, G)
    assert torch.equal(G[0], alone) and vals[0] == v0[0]
    assert vals[1] == 0 and bool((G[1] == 0).all())
    for i in (2, 3):
        assert not bool(torch.isfinite(vals[i])) and not bool(torch.isfinite(G[i]).any())
