"""The planner's run lists (128-tiles of the update list run as 256-tiles) and
the rule that takes fp32 sets to the split form, on the CPU: tests/
run_lists_check.cpp is built with g++ against the planner's own sources."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from workloads import CONFIGS  # noqa: E402

CSRC = os.path.join(ROOT, "paper_2607_08754_amd", "csrc")
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("run_lists") / "run_lists_check")
    cmd = ["g++", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "run_lists_check.cpp"), os.path.join(CSRC, "plan.cpp"),
           os.path.join(CSRC, "pe_schedule.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def run(checker, shapes, dtype, iters=6, coeffs=None, grad=F32, eps=0.0):
    head = f"{dtype} 0 {iters} 0 {1 if coeffs is not None else 0}\n"
    if coeffs is not None:
        head += " ".join(repr(float(c)) for c in coeffs) + "\n"
    body = f"{len(shapes)}\n" + "".join(f"{r} {c}\n" for r, c in shapes) + f"{grad} {eps!r}\n"
    r = subprocess.run([checker], input=head + body, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout[-4000:] + r.stderr[-2000:]
    return dict(kv.split("=") for kv in r.stdout.split()[1:])


@pytest.mark.parametrize("name", sorted(CONFIGS))
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_run_lists(checker, name, dtype):
    got = run(checker, CONFIGS[name].shapes, dtype, CONFIGS[name].iters)
    assert got["split"] == ("1" if dtype == F32 else "0")


def test_run_lists_edges(checker):
    assert run(checker, [(512, 2048)] * 32, F32)["run256"] == "6"       # 512 256-tiles: the smallest such set
    assert run(checker, [(512, 2048)] * 31, F32)["run256"] == "0"
    # dims that are no multiples of 256: edge tiles, while they waste at most a quarter
    for dt in (F32, BF16):
        assert run(checker, [(640, 3456)] * 32, dt)["run256"] == "6"    # 3 x 14 tiles for 2.5 x 13.5
        assert run(checker, [(384, 3200)] * 64, dt)["run256"] == "0"    # 2 x 13 for 1.5 x 12.5
        assert run(checker, [(3456, 1280), (1280, 1280)] * 8, dt)["run256"] == "6"
    run(checker, [(1, 300), (7, 13), (130, 257), (0, 5)], F32)
    cubic = [1.5, -0.5, 0.0] * 6
    assert run(checker, [(512, 2048)] * 32, F32, coeffs=cubic)["run256"] == "0"


# the range rule of the split form: |X| <= 3.5, |B| <= 58 and linear terms that
# leave at least half of X_0 over the whole
# table (twice |B| in the first step, whose matrix is scaled by kappa < 2)
@pytest.mark.parametrize("coeffs,split", [
    ([15 / 8, -10 / 8, 3 / 8] * 2, 1),          # Newton-Schulz
    ([3.4445, -4.7750, 2.0315] * 3, 1),         # maps [0, 1] into [0, 1.3]
    ([1.5, -0.5, 0.0] * 2, 1),                  # cubic
    ([3.4, 0.0, 0.0, 0.2, 0.0, 0.0], 1),        # X up to 3.4
    ([3.6, 0.0, 0.0, 0.2, 0.0, 0.0], 0),        # X up to 3.6
    ([28.0, -40.0, 13.0, 1.0, 0.0, 0.0], 0),    # an interior extremum of X beyond the range
    ([30.0, -100.0, 71.0, 1.0, 0.0, 0.0], 0),   # 2 |B| up to 60 at x = 0
    ([1.0, 0.0, 0.0, 1.0, 60.0, -61.0], 0),     # interior extrema in a later step
    ([0.6, 0.0, 0.0, 2.0, 0.0, 0.0], 1),        # shrinks X, not below half
    ([0.4, 0.0, 0.0, 2.5, 0.0, 0.0], 0),        # below half in the first step
    ([0.6, 0.0, 0.0, -0.6, 0.0, 0.0, 3.0, 0.0, 0.0], 0),   # over two steps
    ([2.0, 0.0, 0.0, 0.2, 0.0, 0.0], 0),        # at the end
    ([0.0, 1.0, 0.0, 2.0, 0.0, 0.0], 0),        # no linear term
])
def test_split_rule(checker, coeffs, split):
    assert run(checker, [(64, 96)], F32, iters=len(coeffs) // 3, coeffs=coeffs)["split"] == str(split)
    assert run(checker, [(64, 96)], BF16, iters=len(coeffs) // 3, coeffs=coeffs)["split"] == "0"


@pytest.mark.parametrize("shapes", [[(200, 300)] * 3, [(100, 256)] * 4, [(512, 2048)] * 32])
@pytest.mark.parametrize("iters", [1, 5, 6, 12])
def test_scales_at_large_eps(checker, shapes, iters):
    """eps > 0 on the split form: every iterate held in the power of two that its
    bound allows, the schedule's value that of the table at X_0 2^-h."""
    run(checker, shapes, F32, iters=iters, eps=0.5)
    run(checker, shapes, BF16, iters=iters, eps=0.5)
    run(checker, shapes, F32, iters=iters, eps=0.5, coeffs=[15 / 8, -10 / 8, 3 / 8] * iters)
    run(checker, shapes, F32, iters=iters, eps=0.5, coeffs=[1.5, -0.5, 0.0] * iters)
    run(checker, shapes, F32, iters=iters, eps=0.5, grad=BF16)


def test_split_needs_fp32_gradients(checker):
    """bf16 gradients of fp32 weights stay on fp32 MFMA, on 128-tiles."""
    got = run(checker, [(512, 2048)] * 32, F32, grad=BF16)
    assert got["split"] == "0" and got["run256"] == "0"


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_short_rule(checker, dtype):
    """One launch per step: every matrix at most 128 x 1024, quintic steps."""
    def short(*args, **kw):
        return run(checker, *args, **kw)["short"] == "1"

    for iters in (1, 2, 5, 6):
        assert short([(128, 256)] * 4, dtype, iters=iters)
    assert short([(1, 7), (1024, 128), (0, 5), (100, 1000)], dtype)
    assert not short([(128, 256), (129, 256)], dtype) and not short([(128, 1025)], dtype)
    assert not short([(0, 5)], dtype) and not short([], dtype)
    assert not short([(128, 256)], dtype, coeffs=[1.5, -0.5, 0.0] * 6)
    assert not short([(128, 256)], dtype, coeffs=[2.0, -1.5, 0.5] * 5 + [1.5, -0.5, 0.0])
    assert short([(128, 256)], dtype, coeffs=[15 / 8, -10 / 8, 3 / 8] * 6)
    assert short([(128, 128)] * 1600, dtype) and not short([(128, 128)] * 1601, dtype)   # partials read a step
    # the partials must not take a set out of the 64 MiB static scratch: 1 MiB
    # of each 128 x 1024 matrix, beside 1.625 (fp32) or 0.8125
    few, at_limit = (20, 25) if dtype == F32 else (25, None)
    assert short([(128, 1024)] * few, dtype)
    if at_limit:
        assert not short([(128, 1024)] * at_limit, dtype)


def test_no_short_steps_on_fp32_mfma(checker):
    assert run(checker, [(128, 256)] * 4, F32, grad=BF16)["short"] == "0"


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_small_tiles(checker, dtype):
    """Symmetric outputs on 64-tiles: at most 512 of them and no XCD's queue with a
    second round (510 equal tiles of 51 matrices: 70 on the longest queue, which
    holds 64); a split Gram product stays on its parts; not on fp32 MFMA."""
    def small(*args, **kw):
        return run(checker, *args, **kw)["small"]

    assert small([(200, 3000)] * 4, dtype) == "01"
    assert small([(200, 250)] * 48, dtype)[1] == "1"                              # 480 64-tiles, queues of 60
    if dtype == BF16:
        assert small([(200, 250)] * 48, dtype) == "11"
    assert small([(200, 250)] * 51, dtype) == "00"                                # 510, queues of up to 70
    assert small([(640, 1920)] * 9, dtype)[1] == "0"                              # 495
    for k in range(40, 53):                                                       # mixed sets around the limit
        small([(200, 250 + 31 * i) for i in range(k)] + [(60, 700)] * (52 - k), dtype)
    assert small([(1, 130), (7, 13), (0, 5), (150, 200)], dtype)[1] == "1"
    assert small([(0, 5)], dtype) == "00"


@pytest.mark.parametrize("dtype,shapes", [
    (BF16, [(512, 1792)] * 10 + [(128, 1792)]),
    # short matrices, whose partials must not hide that the set fits without the lists
    (F32, [(128, 128)] * 151 + [(128, 1024)] * 4 + [(0, 5)] * 120),
    (F32, [(128, 128)] * 147 + [(128, 384)] * 10 + [(0, 5)] * 130),
])
def test_sets_that_fit_the_scratch_without_64_tiles(checker, dtype, shapes):
    """A set that the no-allocation entry's 64 MiB hold without the 64-tile lists
    goes without them."""
    got = run(checker, shapes, dtype)
    assert int(got["ws"]) <= 64 << 20 and got["lean"] == "1" and got["small"] == "00" and got["short"] == "0"


def test_no_small_tiles_on_fp32_mfma(checker):
    assert run(checker, [(200, 250)] * 4, F32, grad=BF16)["small"] == "00"
