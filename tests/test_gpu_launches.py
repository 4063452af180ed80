"""Which kernel a batch's forward and reverse steps run on, for the sizes and
options that the kernels' own tests use, so that none of them passes on another
kernel: the latency kernel with its rows streamed and in both register tiles,
with slabs that read each other directly (at most 64) and through owners, the
kernels of shared tensors, on chip, wave and linear, and the streaming kernel,
whose resident form a mixed batch still reaches."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS = 44100.0, 150


@pytest.fixture(scope="module")
def modal():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    return modal


def _modes(rng, n):
    x0 = 1e-3 * rng.normal(size=n)
    return dict(omega=2 * np.pi * np.sort(rng.uniform(80, 7000, n)), gamma=rng.uniform(1, 30, n), x0=x0, xm1=x0.copy(),
                c=rng.normal(size=n))


def _plate(n, n_in, classed=False):
    rng = np.random.default_rng(n * 1000 + n_in)
    H = rng.normal(size=(n_in, n, n))
    H = 0.5 * (H + H.transpose(0, 2, 1)) * np.sqrt(4.0 / (n * n_in))
    p = dict(_modes(rng, n), kind="vk")
    if classed:
        cls = (np.arange(n) % 4).astype(np.uint8)
        for i in range(n_in):
            H[i] *= (cls[:, None] ^ cls[None, :]) == i % 4
        p["mode_class"] = cls
    return dict(p, Ht=(3e6 * H).astype(np.float32))


def _tension(n):
    return dict(_modes(np.random.default_rng(n), n), kind="tension", lam=np.arange(1.0, n + 1), kappa=1e5)


def _linear(n):
    return dict(_modes(np.random.default_rng(n), n), kind="linear")


def _launches(modal, insts, flags=0, **kw):
    sim = modal.Sim(insts, FS, flags=flags, **kw)
    v = sim.launches()
    sim.close()
    return v


# shapes, slabs of the largest instance, blocks a wave in registers (the 72/9
# plate stays whole: 54 blocks, 7 a wave)
@pytest.mark.parametrize("shapes,slabs,blocks", [
    ([(65, 3)], 1, 4), ([(65, 66)], 33, 4), ([(72, 72)], 18, 4), ([(72, 9), (68, 33), (97, 64)], 32, 8),
    ([(100, 101)], 51, 4), ([(128, 128)], 64, 4), ([(131, 129)], 129, 4), ([(196, 130)], 130, 8), ([(256, 65)], 65, 8),
    ([(257, 40)], 40, 0), ([(66, 5)] * 18, 1, 4)])
def test_latency(modal, shapes, slabs, blocks):
    plates = [_plate(*s) for s in shapes]
    v = _launches(modal, plates)
    assert (v["kernel"], v["instance_workgroups"], v["tile"], v["reverse"]) == ("latency", slabs, blocks, None)
    v = _launches(modal, plates, modal.FLAG_GRAD)
    assert v["kernel"] == "latency"
    assert v["reverse"] == ("latency" if blocks else "resident")


def test_the_other_kernels(modal):
    p = _plate(24, 16, True)
    assert _launches(modal, [p])["kernel"] == "on-chip"
    v = _launches(modal, [p] * 300, modal.FLAG_GRAD)
    assert (v["kernel"], v["workgroups"], v["reverse"], v["reverse_workgroups"]) == ("on-chip", 300, "on-chip", 300)
    v = _launches(modal, [p] * 20)
    assert (v["kernel"], v["workgroups"]) == ("shared by class", 2)
    assert _launches(modal, [_plate(24, 16)] * 20)["kernel"] == "shared"
    v = _launches(modal, [_tension(12)] * 9, modal.FLAG_GRAD)
    assert (v["kernel"], v["workgroups"], v["reverse"]) == ("wave", 3, "wave")
    assert _launches(modal, [_linear(9)])["kernel"] == "linear"
    v = _launches(modal, [_plate(72, 30)], modal.FLAG_GRAD, waves=4, max_workgroups=8)
    assert (v["kernel"], v["reverse"]) == ("streaming", "streaming")
    sim = modal.Sim([p], FS, flags=modal.FLAG_GRAD)
    sim.set_tangent(0, p["Ht"])
    assert sim.launches()["reverse"] in ("streaming", "resident")
    sim.close()


def test_resident_streaming_kernel_of_a_mixed_batch(modal):
    """Beside a tension instance a large plate steps on the streaming kernel
    with resident state, forward and reverse: FP32 forces as on an explicit
    launch shape, so 1e-5."""
    import torch
    insts = [_plate(72, 50), _tension(20), _plate(90, 33)]
    g = torch.tensor(np.random.default_rng(1).normal(size=(3, STEPS)), dtype=torch.float32, device="cuda")
    got = []
    for kw in ({}, dict(waves=4, max_workgroups=24)):
        sim = modal.Sim(insts, FS, flags=modal.FLAG_GRAD, **kw)
        v = sim.launches()
        assert (v["kernel"], v["reverse"]) == (("resident",) * 2 if not kw else ("streaming",) * 2)
        assert kw or v["instance_workgroups"] > 1
        y = sim.run(STEPS).cpu().numpy()
        sim.reset()
        assert np.array_equal(np.concatenate([sim.run(k).cpu().numpy() for k in (1, 49, 100)], 1), y)
        res = sim.grad(STEPS, g)
        got.append([y] + [np.concatenate([np.ravel(a) for a in res[k]]) for k in ("omega", "gamma", "c", "x0", "row")])
        sim.close()
    for a, b in zip(*got):
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b)
