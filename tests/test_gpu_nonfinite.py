"""Infinities and NaN in a field: a run in moments is finite wherever steps with
the collision operator are, with their values, and the dense fractional term
keeps them to the outputs their line reaches, for every choice of tiles."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("value", [np.inf, np.nan], ids=["inf", "nan"])
@pytest.mark.parametrize("dim,n,at", [(2, [70, 45], (20, 31)), (2, [66, 9], (1, 64)), (3, [24, 19, 21], (7, 1, 13))])
def test_a_run_spreads_them_no_further_than_the_operator(dim, n, at, value):
    from paper_1706_09161_amd import LbmFade

    print(f"[gpu-nonfinite] {n} {value}", flush=True)
    cfg = synth.small(dim, n, seed=101, c_wall=0.2, p=[1.0, 0.4, 0.0][:dim])
    good = synth.initial_C(cfg).astype(np.float32)
    bad = good.copy()
    bad[at] = value

    def run(C0, pieces, keep):
        with LbmFade.from_config(cfg, precision="fp32") as s:
            s.set_register_kernels(keep)
            s.set_C(C0)
            for k in pieces:
                s.step(k)
            return s.get_C(device=False), s.get_f(device=False)

    for steps in (1, 4, 6):
        moments, op = run(bad, [steps], False), run(bad, [1] * steps, True)
        clean = run(good, [1] * steps, True)
        for got, ref, fin in zip(moments, op, clean):
            assert np.isfinite(fin).all()
            assert np.isfinite(got)[np.isfinite(ref)].all()
            assert (~np.isfinite(got)).any()
            same = np.isfinite(ref)
            assert np.allclose(got[same], ref[same], rtol=0, atol=1e-5 * np.abs(fin).max())


SIZES = [([333, 300], [0.4, 1.0]), ([768, 760], [0.0, 0.5]), ([120, 128, 127], [1.0, 0.3, 0.0]),
         ([193, 160, 131], [0.3, 1.0, 0.6])]


@pytest.mark.parametrize("n,p,axis", [(n, p, axis) for n, p in SIZES for axis in range(len(n))],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
def test_every_choice_of_tiles_keeps_them_to_their_lines(n, p, axis):
    """n picks the tiles: one output tile and chunks of 128 or 64, two tiles, four."""
    from paper_1706_09161_amd import LbmFade

    dim = len(n)
    print(f"[gpu-nonfinite] {n} axis {axis}", flush=True)
    cfg = synth.small(dim, n, alpha=[1.4] * dim, p=p, seed=102)
    good = np.random.default_rng(103).uniform(0.5, 1.0, synth.shape(cfg)).astype(np.float32)
    bad = good.copy()
    ax = dim - 1 - axis  # array axis of coordinate `axis`
    spots = []
    for k, v in enumerate((np.inf, -np.inf, np.nan)):
        i = [(5 + 11 * k) % m for m in good.shape]
        i[ax] = good.shape[ax] // 2 - 17 + 5 * k
        spots.append((tuple(i), v))
        bad[tuple(i)] = v
    with LbmFade.from_config(cfg, precision="fp32") as s:
        ref = s.apply_phi(torch.from_numpy(good).cuda())[axis].cpu().numpy()
        got = s.apply_phi(torch.from_numpy(bad).cuda())[axis].cpu().numpy()
    want, redone = ref.copy(), np.zeros(ref.shape, bool)
    for i, v in spots:
        line = tuple(slice(None) if a == ax else i[a] for a in range(dim))
        redone[line] = True
        j, w = np.arange(good.shape[ax]), want[line].copy()
        reach = np.ones(j.size, bool) if 0 < p[axis] < 1 else (j >= i[ax] if p[axis] == 1.0 else j <= i[ax])
        w[reach] = v
        want[line] = w
    assert np.array_equal(got[~redone], ref[~redone])
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)])
    # rounded sums of up to 768 products of values of one sign, taken one by one
    assert np.allclose(got[fin], want[fin], rtol=768 * 2.0**-24, atol=0)
