"""The fractional term of long axes (near band plus moments of far boxes) at
the sizes where it can go wrong: the longest dense axes and the shortest and
longest ones beyond, ends of boxes, ragged ends, few lines, every axis of a
grid, a long axis beside a short one (summed densely with it, or on its own),
one- and two-sided operators; and lines that hold infinities or NaN.

FP32 tolerance, relative to sum_k |K_jk| |C_k| (the value itself: C and every
weight are >= 0): an accumulator of the band is rounded 8 times and the three
of them are added (12 roundings); a moment takes 5 roundings and a local
coefficient at most 8, each passed on through interpolation weights whose
absolute sum is at most 2.8 per box (5 * 2.8^2 + 8 * 2.8 = 62); two more for
the boundary columns; roundings of the matrix cores are within one unit
(2^-23).  76 * 2^-23 in all; the interpolation itself adds less than 1e-10.
Split BF16: 2^-14, as everywhere.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # (dim, n, alpha, p)
    (2, [640, 35], [1.3, 1.5], [0.3, 0.5]),
    (2, [35, 641], [1.5, 1.2], [0.5, 0.8]),
    (2, [703, 768], [1.05, 1.95], [1.0, 0.0]),
    (2, [769, 1023], [1.7, 1.4], [0.0, 1.0]),
    (2, [770, 895], [1.4, 1.6], [0.3, 0.0]),
    (2, [900, 832], [1.6, 1.3], [1.0, 0.6]),
    (2, [1025, 33], [1.2, 1.5], [0.6, 0.5]),
    (2, [3, 1153], [1.5, 1.6], [0.5, 1.0]),
    (2, [1216, 650], [1.9, 1.1], [0.4, 0.0]),
    (2, [4096, 5], [1.2, 1.5], [0.7, 0.5]),
    (2, [40, 4095], [1.5, 1.4], [0.5, 0.0]),
    (3, [9, 855, 4], [1.5, 1.3, 1.5], [0.5, 0.3, 0.5]),
    (3, [5, 7, 1100], [1.5, 1.5, 1.8], [0.5, 0.5, 0.9]),
    (3, [866, 5, 4], [2.0, 1.5, 1.5], [0.5, 0.5, 0.5]),
    # every axis long, or enough lines beside a short axis for a launch of the long one's own
    (2, [1153, 770], [1.5, 1.6], [0.5, 1.0]),
    (2, [4096, 769], [1.2, 1.5], [0.7, 0.0]),
    (2, [771, 4095], [1.5, 1.4], [0.5, 0.0]),
    (3, [866, 64, 45], [2.0, 1.5, 1.5], [0.5, 0.5, 0.5]),
    (3, [24, 1100, 90], [1.5, 1.3, 1.5], [0.5, 0.3, 0.5]),
    (3, [70, 30, 1100], [1.5, 1.5, 1.8], [0.5, 0.5, 0.9]),
]


def _solver(cfg, precision):
    from paper_1706_09161_amd import LbmFade

    return LbmFade.from_config(cfg, precision=precision)


def _config(case, **kw):
    dim, n, alpha, p = case
    cfg = synth.small(dim, n, alpha=alpha, p=p, seed=51, **kw)
    cfg["g"] = [1.3, 0.7, 1.1][:dim]
    cfg["dx"] = 0.5
    return cfg


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[1])))
def test_long_axes_match_oracle(case, precision):
    dim, n, _, _ = case
    print(f"[gpu-far] {precision} {n}", flush=True)
    cfg = _config(case, flux_form="rl")
    C = np.random.default_rng(23).uniform(0.0, 1.0, synth.shape(cfg)).astype(np.float32)
    ref = oracle.phi(cfg, C.astype(np.float64))
    with _solver(cfg, precision) as s:
        out = torch.full((dim,) + tuple(C.shape), float("nan"), device="cuda")
        s.apply_phi(torch.from_numpy(C).cuda(), out=out)
        got = out.cpu().numpy().astype(np.float64)
    tol = 76 * 2.0**-23 if precision == "fp32" else 2.0**-14
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - ref) <= tol * np.abs(ref) + 1e-30), np.max(np.abs(got - ref) / (np.abs(ref) + 1e-30))


@pytest.mark.parametrize("p", [[0.4, 0.5], [1.0, 0.5], [0.0, 0.5]], ids=["two-sided", "left", "right"])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("size", [70, 700, 900])
def test_lines_with_infinities_and_nan(size, axis, p):
    """One line with +inf, one with -inf, one with NaN at an inner node, on
    dense axes and one with boxes: the outputs whose integral reaches the node take its value
    (every weight is > 0) and every other output is that of the finite field."""
    lines = 800 if size == 900 else 40  # boxes: every axis long
    n, at = [size, lines], size // 2 - 17
    pa = list(p)
    if axis == 1:
        n, pa = n[::-1], pa[::-1]
    cfg = synth.small(2, n, alpha=[1.4, 1.4], p=pa, seed=52)
    C = np.random.default_rng(24).uniform(0.5, 1.0, (lines, size)).astype(np.float32)  # [line, node]
    bad = C.copy()
    for line, v in ((3, np.inf), (17, -np.inf), (38, np.nan)):
        bad[line, at] = v

    def lay(a):
        return np.ascontiguousarray(a if axis == 0 else a.T)

    with _solver(cfg, "fp32") as s:
        good = s.apply_phi(torch.from_numpy(lay(C)).cuda())[axis].cpu().numpy()
        got = s.apply_phi(torch.from_numpy(lay(bad)).cuda())[axis].cpu().numpy()
    if axis == 1:
        good, got = good.T, got.T
    j = np.arange(size)
    reach = np.ones(size, bool) if 0 < p[0] < 1 else (j >= at if p[0] == 1.0 else j <= at)
    for line in range(lines):
        want = good[line].copy()
        if line in (3, 17, 38):
            want[reach] = bad[line, at]
        fin = np.isfinite(want)
        assert np.array_equal(np.isnan(got[line]), np.isnan(want)), line
        assert np.array_equal(got[line][~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)]), line
        assert np.allclose(got[line][fin], want[fin], rtol=1e-4, atol=0), line
