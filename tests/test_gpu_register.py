"""Where the dense fractional term runs on the register kernels by itself: the
sizes on both sides of each line.  set_register_kernels keeps axes with far
boxes on them too: on a grid whose axes all have boxes, and where a long axis with boxes lies
beside a short one; and fade_solve, which sets it, there.  The tile that the
size selects, forced, gives the same bits."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILE = "15"  # the register kernel of these sizes: 128 outputs, k in 4 shares, one group of C ahead


def _field(cfg, seed):
    return torch.from_numpy(np.random.default_rng(seed).uniform(0.0, 1.0, synth.shape(cfg)).astype(np.float32)).cuda()


@pytest.mark.parametrize("n", [[900, 800], [4096, 200], [200, 4096]], ids=lambda n: "x".join(map(str, n)))
def test_boxed_axes_stay_on_the_register_kernels(n, monkeypatch):
    from paper_1706_09161_amd import LbmFade

    print(f"[gpu-register] {n}", flush=True)
    cfg = synth.small(2, n, alpha=[1.4, 1.7], p=[0.3, 0.6], seed=81)
    C = _field(cfg, 31)

    def run(keep):
        with LbmFade.from_config(cfg, precision="fp32") as s:
            s.set_register_kernels(keep)
            s.set_C(C)
            s.step(11)
            return s.apply_phi(C), s.get_C()

    default, kept = run(False), run(True)
    monkeypatch.setenv("LBM_FP32_TILE", TILE)
    forced = run(True)
    assert torch.equal(kept[0], forced[0]) and torch.equal(kept[1], forced[1])
    assert not torch.equal(kept[0], default[0])


def test_gradients_on_boxed_axes(monkeypatch):
    from paper_1706_09161_amd.autograd import fade_solve

    cfg = synth.small(2, [800, 780], alpha=[1.4, 1.7], seed=82)
    C0, obs = _field(cfg, 32), _field(cfg, 33)

    def run():
        leaf = [C0.clone().requires_grad_(True)] + [
            torch.tensor(np.asarray(v), dtype=torch.float64, requires_grad=True)
            for v in ([[0.1, 0.02], [0.02, 0.12]], [0.02, -0.01], [0.4, 0.7])]
        C = fade_solve(leaf[0], None, *leaf[1:], alpha=cfg["alpha"], steps=5, ckpt_every=2)
        return [C.detach()] + list(torch.autograd.grad(0.5 * ((C - obs) ** 2).sum(), leaf))

    default = run()
    monkeypatch.setenv("LBM_FP32_TILE", TILE)
    for a, b in zip(run(), default):
        assert torch.equal(a, b)


@pytest.mark.parametrize(
    "precision,n,p,register",
    [("fp32", [64, 64], [0.5, 0.5], False), ("fp32", [72, 64], [0.5, 0.5], True), ("fp32", [128, 128], [1.0, 0.0], True),
     ("fp32", [136, 128], [0.5, 0.5], False), ("fp32", [128, 136], [1.0, 0.0], True),
     ("fp32", [224, 224], [1.0, 0.0], True), ("fp32", [232, 232], [1.0, 0.0], False),
     ("fp32", [232, 232], [1.0, 0.5], True), ("fp32", [384, 384], [0.5, 0.0], True),
     ("fp32", [384, 392], [0.5, 0.5], False), ("fp32", [225, 224], [0.5, 0.5], False),
     ("bf16x3", [384, 384], [0.5, 0.5], False), ("bf16x3", [400, 512], [0.5, 1.0], True),
     ("bf16x3", [400, 512], [0.0, 1.0], False), ("bf16x3", [512, 384], [0.5, 0.5], False),
     ("bf16x3", [96, 512], [0.5, 0.5], True), ("bf16x3", [968, 1000], [0.5, 0.5], True),
     ("bf16x3", [968, 1000], [1.0, 0.0], False), ("bf16x3", [952, 1000], [0.5, 0.5], False),
     ("bf16x3", [1000, 1032], [0.5, 0.5], False),
     ("bf16x3", [528, 528], [0.5, 0.5], False), ("bf16x3", [848, 64], [0.5, 0.5], True),
     ("bf16x3", [848, 16, 16], [0.5, 0.5, 0.5], False)],
    ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
def test_lines_between_the_dense_kernels(precision, n, p, register):
    from paper_1706_09161_amd import LbmFade

    cfg = synth.small(len(n), n, alpha=[1.4, 1.7, 1.5][:len(n)], p=p, seed=83)
    C = _field(cfg, 34)
    with LbmFade.from_config(cfg, precision=precision) as s:
        default = s.apply_phi(C)
        s.set_register_kernels(True)
        kept = s.apply_phi(C)
    assert torch.equal(default, kept) == register
