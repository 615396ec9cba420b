"""The dense fractional term on the BF16 matrix cores (three-term splits for
FP32, the 3-term split for bf16x3) at the sizes where it can go wrong: edges of
output tiles (64, 128, 256), chunks of k (64, 128) and steps of 16, ragged ends,
line blocks that are not full, the smallest boxes, every choice of tiles (few
and many workgroups, 2D and 3D), one- and two-sided operators.

FP32 tolerance, relative to sum_k |K_jk| |C_k| (the value itself: C and every
weight are >= 0): each of the k shares' accumulators is rounded once per 16
products, at most (n + 63) / 64 + 16 / 4 times, and at most 12 sums follow
(shares, correction, boundary columns), all within one unit (2^-23): for
n <= 640, 26 * 2^-23; one wavefront's whole range (many workgroups, n <= 200
here) is at most 13 + 12 roundings.  Split BF16: 2^-14, as everywhere.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # (dim, n, alpha, p)
    (2, [3, 3], [1.5, 1.5], [0.5, 0.5]),
    (2, [15, 17], [1.3, 1.7], [1.0, 0.0]),
    (2, [33, 63], [1.5, 1.2], [0.0, 0.4]),
    (2, [64, 65], [1.4, 1.6], [0.3, 1.0]),
    (2, [127, 129], [1.05, 1.95], [0.5, 0.0]),
    (2, [128, 191], [1.5, 1.8], [1.0, 0.7]),
    (2, [255, 257], [1.2, 1.4], [0.6, 0.0]),
    (2, [513, 385], [1.7, 1.3], [1.0, 0.5]),
    (2, [640, 31], [1.6, 1.5], [0.0, 0.5]),
    (3, [4, 3, 5], [1.5, 1.5, 1.5], [0.5, 1.0, 0.0]),
    (3, [65, 33, 31], [1.5, 1.6, 1.8], [0.5, 0.2, 0.9]),
    (3, [120, 128, 127], [1.3, 1.9, 1.4], [1.0, 0.0, 0.6]),      # two output tiles per workgroup
    (3, [193, 160, 131], [1.4, 1.5, 1.2], [0.3, 1.0, 0.0]),      # four
    (3, [9, 100, 70], [2.0, 1.1, 1.5], [0.5, 0.5, 0.5]),
]


@pytest.mark.parametrize("precision", ["fp32", "bf16x3"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[1])))
def test_dense_axes_match_oracle(case, precision):
    from paper_1706_09161_amd import LbmFade

    dim, n, alpha, p = case
    print(f"[gpu-split] {precision} {n}", flush=True)
    cfg = synth.small(dim, n, alpha=alpha, p=p, seed=61)
    cfg["g"] = [1.3, 0.7, 1.1][:dim]
    cfg["dx"] = 0.5
    C = np.random.default_rng(29).uniform(0.0, 1.0, synth.shape(cfg)).astype(np.float32)
    ref = oracle.phi(cfg, C.astype(np.float64))
    with LbmFade.from_config(cfg, precision=precision) as s:
        out = torch.full((dim,) + tuple(C.shape), float("nan"), device="cuda")
        s.apply_phi(torch.from_numpy(C).cuda(), out=out)
        got = out.cpu().numpy().astype(np.float64)
    tol = 26 * 2.0**-23 if precision == "fp32" else 2.0**-14
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - ref) <= tol * np.abs(ref) + 1e-30), np.max(np.abs(got - ref) / (np.abs(ref) + 1e-30))


@pytest.mark.parametrize("precision,tile", [("fp32", "13"), ("bf16x3", "13")])
def test_register_kernels_can_be_kept(precision, tile, monkeypatch):
    """set_register_kernels keeps a small ragged grid on the register kernel
    that its size selects (the forced tile), also in a replayed step graph,
    and off it goes back to the default."""
    from paper_1706_09161_amd import LbmFade

    cfg = synth.small(2, [61, 45], alpha=[1.4, 1.7], p=[0.3, 0.6], seed=62)
    C = torch.from_numpy(np.random.default_rng(30).uniform(0.0, 1.0, synth.shape(cfg)).astype(np.float32)).cuda()

    def run(s):
        s.set_C(C)
        s.step(23)
        return s.apply_phi(C).cpu().numpy(), s.get_C(device=False)

    with LbmFade.from_config(cfg, precision=precision) as s:
        default = run(s)
        s.set_register_kernels(True)
        kept = run(s)
        s.set_register_kernels(False)
        again = run(s)
    monkeypatch.setenv("LBM_FP32_TILE" if precision == "fp32" else "LBM_BF16_TILE", tile)
    with LbmFade.from_config(cfg, precision=precision) as s:
        forced = run(s)
    assert np.array_equal(kept[0], forced[0])  # (the runs' collisions differ: the switch keeps that of the register kernels too)
    for k in range(2):
        assert np.array_equal(again[k], default[k])
    assert not np.array_equal(kept[0], default[0])  # the two kernels round differently
