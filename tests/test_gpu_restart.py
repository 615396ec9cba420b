"""A run continued in another handle from saved populations and concentration
(get_f and get_C, then set_f with both) gives the bits of the run they were
saved from, wherever it was cut.  Saved populations alone do the same where C
is their sum (BGK, MRT with other free relaxation times, and the register
kernels' collision); elsewhere set_f brings C back to the rounding of f."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # (dim, n, collision, free relaxation time, source, space-dependent fields, precision)
    (2, [64, 64], "MRT", 1.0, False, False, "fp32"),
    (2, [130, 67], "MRT", 1.0, True, True, "fp32"),
    (2, [75, 58], "MRT", 1.0, True, False, "bf16x3"),
    (2, [600, 450], "MRT", 1.0, False, False, "fp32"),
    (2, [75, 58], "MRT", 0.8, True, False, "fp32"),
    (2, [75, 58], "BGK", 1.0, True, False, "fp32"),
    (3, [24, 19, 21], "MRT", 1.0, True, False, "fp32"),
    (3, [65, 9, 4], "MRT", 1.0, False, True, "fp32"),
    (3, [24, 19, 21], "BGK", 1.0, False, False, "fp32"),
]


@pytest.mark.parametrize("keep", [False, True], ids=["default", "register"])
@pytest.mark.parametrize("dim,n,collision,tau,with_source,var,precision", CASES)
def test_continues_from_saved_populations(dim, n, collision, tau, with_source, var, precision, keep):
    from paper_1706_09161_amd import LbmFade

    print(f"[gpu-restart] dim={dim} n={n} {collision} tau={tau} var={var} {precision} keep={keep}", flush=True)
    kw = dict(D=(0.1 * np.eye(dim)).tolist()) if collision == "BGK" else {}
    cfg = synth.small(dim, n, seed=71, with_source=with_source, c_wall=0.3, collision=collision, tau_free=[tau] * 4, **kw)
    C0 = synth.initial_C(cfg).astype(np.float32)

    def handle():
        s = LbmFade.from_config(cfg, precision=precision)
        s.set_register_kernels(keep)
        if with_source:
            s.set_source(synth.source(cfg).astype(np.float32))
        if var:
            s.set_diffusion(synth.random_tensor_field(cfg, seed=72).astype(np.float32))
            s.set_wall(synth.random_wall_values(cfg, seed=73).astype(np.float32))
        return s

    with handle() as s:
        s.set_C(C0)
        s.step(31)
        ref_f, ref_C = s.get_f(device=False), s.get_C(device=False)
    summed = keep or collision == "BGK" or tau != 1.0
    for cut, device in ((0, True), (1, False), (7, True), (20, False)):
        with handle() as s:
            s.set_C(C0)
            s.step(cut)
            f, C = s.get_f(device=device), s.get_C(device=device)
        for given in (C, None) if summed else (C,):
            with handle() as s:
                s.set_f(f, C=given)
                assert np.array_equal(s.get_C(device=False), C.cpu().numpy() if device else C), cut
                s.step(31 - cut)
                assert np.array_equal(s.get_f(device=False), ref_f), cut
                assert np.array_equal(s.get_C(device=False), ref_C), cut
        if not summed:
            with handle() as s:
                s.set_f(f)
                off = s.get_C(device=False) - (C.cpu().numpy() if device else C)
            # the moment of f is C to the rounding of f
            assert np.abs(off).max() <= 4 * 2.0**-24 * (2 * dim + 1) * float(abs(f).max()), cut


def test_state_arguments():
    from paper_1706_09161_amd import LbmFade

    cfg = synth.small(2, [24, 20], seed=74)
    with LbmFade.from_config(cfg, precision="fp32") as s:
        s.set_C(synth.initial_C(cfg).astype(np.float32))
        f, C = s.get_f(), s.get_C()
        with pytest.raises(ValueError):
            s.set_f(f, C=C.cpu().numpy())
        with pytest.raises(ValueError):
            s.set_f(f, C=C[1:])
