"""fp32 sets iterated in split form (two fp16 numbers per value) against the
oracle at the edges of its tiles, the 256-tile kernels against 64-bit torch;
the ends of the form's range (tiny norms, eps far above the norm, a row that
carries the norm); and tables outside it, which keep fp32 MFMA."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from oracle.pe_schedule import default_table  # noqa: E402
from parity_util import compare, exact64, run_gpu, run_oracle  # noqa: E402
from workloads import gaussian  # noqa: E402

pytestmark = pytest.mark.gpu

# rows and columns around the 32-value runs, the 64-column wave tiles and the
# 128-tiles; single rows; a long thin one (split-K Gram)
EDGES = [(31, 33), (32, 32), (33, 31), (64, 65), (127, 129), (128, 256), (1, 40), (65, 4100), (385, 384)]


@pytest.mark.parametrize("iters", [5, 6])
def test_split_edges(iters):
    """fp32 tolerance (1e-4) on every measure; the values to 2e-6: T steps of
    fp32 accumulation (rounding 2^-24 per 16 terms) scaled by the unconverged
    last polynomial's slope, about 10 at T = 5."""
    arrs = [gaussian(s, seed=60, std=0.05, dtype="f32", index=i) for i, s in enumerate(EDGES)]
    stationary = [min(s) == 1 for s in EDGES]
    vals, grads, _ = run_gpu(arrs, "f32", "hoyer", iters)
    refs = run_oracle(arrs, "f32", "hoyer", iters)
    compare(vals, grads, refs, "hoyer", "f32", label=f"split edges T={iters}", stationary=stationary)
    assert max(abs(vals[i] - r.value) / r.value for i, r in enumerate(refs)) <= 2e-6


@pytest.mark.parametrize("shape,n", [((512, 2048), 32), ((2048, 512), 32)])
def test_split_256_tiles(shape, n):
    """The smallest set whose update runs on 256-tiles: every matrix against
    the same iteration in float64."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(9)
    W = [torch.randn(shape, generator=gen, device="cuda:0") * 0.02 for _ in range(n)]
    G = [torch.empty(shape, device="cuda:0") for _ in range(n)]
    plan = Plan([shape] * n, dtype="f32", iters=6)
    assert any(op == "update" and edge == 256 for op, _, edge in plan.launches())
    vals = plan(W, G).double()
    for i, w in enumerate(W):
        w = w.double()
        y = w if shape[0] <= shape[1] else w.t().contiguous()
        f = y.norm()
        x = y / f
        for a, b, c in default_table(6):
            s = x @ x.t()
            x = a * x + (b * s + c * (s @ s)) @ x
        nh = (y * x).sum()
        g = 2 * nh / f ** 2 * x - 2 * nh ** 2 / f ** 4 * y
        g = g if shape[0] <= shape[1] else g.t()
        assert abs(vals[i] - (nh / f) ** 2) <= 1e-6 * (nh / f) ** 2, i
        assert (G[i] - g).norm() <= 2e-5 * g.norm(), i


def test_split_256_tiles_of_symmetric_outputs():
    """The smallest set (by matrices of this shape) whose poly products run on
    256-tiles: 520 upper ones. Every tenth matrix against the iteration in
    float64, at the bars of test_split_256_tiles."""
    import torch
    from paper_2607_08754_amd import Plan
    shapes = [(1024, 2048)] * 52
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(13)
    W = [torch.randn(s, generator=gen, device="cuda:0") * 0.02 for s in shapes]
    G = [torch.full(s, float("nan"), device="cuda:0") for s in shapes]
    plan = Plan(shapes, dtype="f32", iters=6)
    assert {"k_tile<gram, 256x256>", "k_tile<poly, 256x256>", "k_upd256<update>"} <= {k for k, _ in plan.kernels()}
    vals = plan(W, G).double()
    for i in range(0, len(W), 10):
        v, g = exact64(W[i], "hoyer", default_table(6))
        assert abs(vals[i] - v) <= 1e-6 * v, i
        assert (G[i] - g).norm() <= 2e-5 * g.norm(), i
    assert all(bool(torch.isfinite(x).all()) for x in G)


def test_table_outside_the_split_range():
    """An explicit table whose iterate reaches 16 (65536 in fp16's scale)."""
    table = np.array([[16.0, 0.0, 0.0], [1 / 16, 0.0, 0.0], [1.875, -1.25, 0.375]])
    shapes = [(80, 150), (150, 80)]
    arrs = [gaussian(s, seed=22, std=1.0, dtype="f32", index=i) for i, s in enumerate(shapes)]
    vals, grads, _ = run_gpu(arrs, "f32", "nuclear", 3, coeffs=table)
    refs = run_oracle(arrs, "f32", "nuclear", 3, table=table)
    compare(vals, grads, refs, "nuclear", "f32", label="outside the split range")


@pytest.mark.parametrize("kind", ["hoyer", "nuclear"])
def test_tiny_norms(kind):
    """Norms down to 2^-125, down to the last bit of fp32's smallest numbers:
    the iterate's scale times 2^-e exceeds fp32's range from 2^-115. The scaling
    is by powers of two and so exact: bit for bit the results of the unscaled
    weights (Hoyer's gradient grows by the inverse and leaves fp32: values)."""
    shapes = [(100, 200), (300, 130), (384, 1536)]
    # 8 significand bits, so that the scaled values are exact
    arrs = [(np.round(gaussian(s, seed=23, std=1.0, dtype="f32", index=i) * 64) / 4096).astype(np.float32)
            for i, s in enumerate(shapes)]
    v0, g0, _ = run_gpu(arrs, "f32", kind, 6)
    for k in (-100, -118, -126):
        small = [np.ldexp(a, k).astype(np.float32) for a in arrs]
        assert all(np.array_equal(np.ldexp(s.astype(np.float64), -k), a) for s, a in zip(small, arrs))
        v1, g1, _ = run_gpu(small, "f32", kind, 6)
        n = len(shapes)
        assert np.array_equal(v1[:n], v0[:n] * (2.0 ** k if kind == "nuclear" else 1.0)), k
        if kind == "nuclear":
            for a, b in zip(g1, g0):
                assert np.array_equal(a, b), k


# per product with one tile of rows and with several, a launch per step, a
# split Gram product, 256-tile updates
@pytest.mark.parametrize("shapes", [[(100, 200), (128, 1000)], [(384, 1536), (300, 130)], [(100, 4000), (700, 300)],
                                    [(512, 2048)] * 32])
@pytest.mark.parametrize("kind", ["hoyer", "nuclear"])
def test_eps_above_the_norm(shapes, kind):
    """eps up to 1e8 times the norm: X_0 is small against 1, and the iterate is
    held in powers of two that keep its significand. 8e-6 and 1e-6 as at eps = 0,
    where these matrices are off by up to 5.4e-6 (Hoyer's difference of two terms);
    less above, where B is a I and little else."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(41)
    W = [torch.randn(s, generator=gen, device="cuda:0") * 0.02 for s in shapes]
    f = [float(w.double().norm()) for w in W]
    table = default_table(6)
    for r in (1e-2, 1.0, 3.0, 1e2, 1e3, 1e4, 1e5, 1e6, 1e8):
        eps = float(np.float32(r * min(f)))
        G = [torch.full(s, float("nan"), device="cuda:0") for s in shapes]
        vals = Plan(shapes, dtype="f32", kind=kind, eps=eps)(W, G).double()
        worst = [0.0, 0.0]
        for i in (0, 1):
            v, g = exact64(W[i], kind, table, eps)
            worst[0] = max(worst[0], float((G[i].double() - g).norm() / g.norm()))
            worst[1] = max(worst[1], float(abs(vals[i] - v) / v))
        print(f"{shapes[0]} {kind} eps/f {r:g}: gradient {worst[0]:.1e} value {worst[1]:.1e}", flush=True)
        assert worst[0] <= 8e-6 and worst[1] <= 1e-6, r


@pytest.mark.parametrize("shrink", [0.4, 1e-2, 1e-4])
def test_table_that_shrinks_the_iterate(shrink):
    """An explicit table whose first step shrinks the iterate and whose next two
    restore it: 3e-6, ten times the 2.6e-7 of fp32 MFMA's sums at T = 4."""
    back = shrink ** -0.5
    table = np.array([[shrink, 0.0, 0.0], [back, 0.0, 0.0], [back, 0.0, 0.0], [1.875, -1.25, 0.375]])
    if back > 50:
        table[1:3, 0] = 50.0
    shapes = [(200, 300), (300, 200), (100, 600)]
    arrs = [gaussian(s, seed=27, std=1.0, dtype="f32", index=i) for i, s in enumerate(shapes)]
    vals, grads, _ = run_gpu(arrs, "f32", "nuclear", 4, coeffs=table)
    refs = run_oracle(arrs, "f32", "nuclear", 4, table=table)
    for i, r in enumerate(refs):
        ge = np.linalg.norm(grads[i] - r.grad) / np.linalg.norm(r.grad)
        print(f"shrink {shrink} {shapes[i]}: gradient {ge:.1e}", flush=True)
        assert ge <= 3e-6 and abs(vals[i] - r.value) <= 1e-6 * r.value, i


@pytest.mark.parametrize("factor", [1e2, 1e3, 1e5])
def test_dominant_row(factor):
    """One row carries the norm: the other rows lie close to the split form's
    smallest value, 2^-36 of the norm's power of two. X, A and B are each rounded
    to it (2^-36 / sqrt(12) a value), and the steps amplify that 2.3e3 times; three
    of those beside the ordinary 8e-6."""
    import torch
    from paper_2607_08754_amd import Plan
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(43)
    for shape in [(384, 1536), (3000, 700)]:
        w = torch.randn(shape, generator=gen, device="cuda:0") * 0.02
        (w if shape[0] < shape[1] else w.t())[3] *= factor
        G = torch.full(shape, float("nan"), device="cuda:0")
        vals = Plan([shape], dtype="f32", kind="nuclear")([w], [G]).double()
        v, g = exact64(w, "nuclear", default_table(6))
        ge = float((G.double() - g).norm() / g.norm())
        print(f"{shape} row {factor:g}: gradient {ge:.1e}", flush=True)
        floor = 2.3e3 * 2.0 ** -36 * (shape[0] * shape[1] / 12) ** 0.5 / float(g.norm())
        assert ge <= 8e-6 + 3 * floor
        assert abs(vals[0] - v) <= 2e-6 * v
