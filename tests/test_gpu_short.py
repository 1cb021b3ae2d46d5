"""Sets of short matrices (at most 128 x 1024), one launch per step, against the
iteration in float64 and against the same matrices beside a wider one, which
takes the set through a launch per product."""
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


# one slice; two; the most; edges inside a slice; tall; one row, one element
SHAPES = [(128, 128), (128, 256), (100, 1024), (1000, 128), (33, 130), (129, 17), (1, 300), (1, 1), (64, 900)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kind,iters", [("hoyer", 5), ("nuclear", 6), ("nuclear", 1), ("hoyer", 7)])
def test_short_sets(dtype, kind, iters):
    """The parity bars (bf16: 2e-2, fp32: 1e-4; after 5 steps the value of a single
    row still has a slope of about 5 in it, 5 x 2^-11 a rounding); and the set's
    error is that of a launch per product (25 % for the chance of one draw of
    roundings)."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(29)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    W = [(torch.randn(s, generator=gen, device="cuda:0") * 0.02).to(dt) for s in SHAPES]
    wide = (torch.randn(200, 300, generator=gen, device="cuda:0") * 0.02).to(dt)
    got = []
    for ws in (W, W + [wide]):
        G = [torch.full(w.shape, float("nan"), device="cuda:0") for w in ws]
        plan = Plan([tuple(w.shape) for w in ws], dtype=dtype, kind=kind, iters=iters)
        for _ in range(3):                       # replays of the captured graph
            vals = plan(ws, G)
        got.append((vals.double(), G))
    table = default_table(iters)
    gtol = vtol = 2e-2 if dtype == "bf16" else 1e-4
    err, size = [0.0, 0.0], 0.0
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
    print(f"one launch per step {err[0]:.3e} per product {err[1]:.3e}", flush=True)
    assert err[0] <= 1.25 * err[1]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_short_options(dtype):
    """Values only, deferred and accumulated gradients agree with the plain call
    bit for bit; without a graph too; NaN, zero and empty matrices stay their own."""
    import torch
    from paper_2607_08754_amd import Plan
    shapes = [(100, 400), (0, 5), (256, 128), (60, 61), (128, 700)]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(31)
    W = [(torch.randn(s, generator=gen, device="cuda:0") * 0.02).to(dt) for s in shapes]

    def call(**kw):
        G = [torch.full(s, 0.5 if kw.get("accumulate") else float("nan"), device="cuda:0") for s in shapes]
        p = Plan(shapes, dtype=dtype, **kw)
        v = p(W) if kw.get("values_only") or kw.get("defer_grad") else p(W, G)
        if kw.get("defer_grad"):
            p.grad(W, G)
        return v.clone(), G

    v, G = call()
    for kw in ({"values_only": True}, {"graph": False}, {"defer_grad": True}, {"accumulate": True}):
        v2, G2 = call(**kw)
        assert torch.equal(v, v2), kw
        for g, g2 in zip(G, G2):
            if kw.get("accumulate"):
                assert torch.equal(g2, g + 0.5)
            elif not kw.get("values_only"):
                assert torch.equal(g, g2), kw
    W[0][3, 5] = float("nan")
    W[3].zero_()
    v3, G3 = call()
    assert bool(torch.isnan(v3[0])) and v3[3] == 0 and bool((G3[3] == 0).all())
    for i in (2, 4):
        assert v3[i] == v[i] and torch.equal(G3[i], G[i])


@pytest.mark.parametrize("shapes", [[(128, 256)] * 4, [(384, 1536)] * 48])
def test_profiled_entries_without_a_kernel(shapes):
    """A profiled call times the kernels that run; entries that run nothing (the
    products of a step that runs as one kernel, the reduce of a Gram product of
    one part per tile) take 0 ms; the results are the call's."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(37)
    W = [torch.randn(s, generator=gen, device="cuda:0") * 0.02 for s in shapes]
    G = [[torch.empty(s, device="cuda:0") for s in shapes] for _ in range(2)]
    plan = Plan(shapes, dtype="f32")
    v = plan(W, G[0]).clone()
    v2, launches = plan.profiled(W, G[1])
    assert torch.equal(v, v2) and all(torch.equal(a, b) for a, b in zip(*G))
    kernels = plan.kernels()
    assert len(launches) == len(kernels) and any(not k for k, _ in kernels)
    for (op, ms), (k, _) in zip(launches, kernels):
        assert (ms > 0.0) if k else (ms == 0.0), (op, k, ms)
