"""A reset that a caller captured: its replay puts the state and the step
counter back, so the next eager run plays the excitation from its start, on
every path that keeps a state."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS = 44100.0, 60


def _instance(kind, n, n_in):
    rng = np.random.default_rng(n)
    x0 = 1e-3 * rng.normal(size=n)
    p = dict(kind=kind, omega=2 * np.pi * np.linspace(80, 7000, n), gamma=np.full(n, 5.0), x0=x0, xm1=x0.copy(),
             c=rng.normal(size=n), b_ext=20 * rng.normal(size=n), e_ext=rng.normal(size=2 * STEPS).astype(np.float32))
    if kind == "vk":
        H = rng.normal(size=(n_in, n, n))
        p["Ht"] = (1e4 * (H + H.transpose(0, 2, 1))).astype(np.float32)
    else:
        p["lam"], p["kappa"] = np.arange(1.0, n + 1), 1e5
    return p


@pytest.mark.parametrize("path", ["wave", "on-chip", "latency", "streaming", "shared", "shared by class"])
def test_replayed_reset(path):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    kw = dict(waves=4, max_workgroups=8) if path == "streaming" else {}
    insts = {"wave": [_instance("tension", 12, 0)] * 5, "on-chip": [_instance("vk", 20, 9)] * 2,
             "latency": [_instance("vk", 80, 20)], "streaming": [_instance("vk", 40, 20)]}.get(path)
    if insts is None:
        p = _instance("vk", 20, 8)
        if path == "shared by class":
            cls = (np.arange(20) % 4).astype(np.uint8)
            keep = (cls[:, None] ^ cls[None, :]) == 1
            p = dict(p, Ht=(p["Ht"] * keep).astype(np.float32), mode_class=cls)
        insts = [p] * 32
    stream = torch.cuda.Stream()
    sim = modal.Sim(insts, FS, flags=modal.FLAG_ASYNC, stream=stream, **kw)
    assert sim.launches()["kernel"] == path
    y = [torch.empty((len(insts), STEPS), device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    sim.run(STEPS, out=y[0])
    sim.run(STEPS, out=y[1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sim.reset()
    for _ in range(2):
        with torch.cuda.stream(stream):
            graph.replay()
        sim.run(STEPS, out=y[2])
        sim.run(STEPS, out=y[3])
        sim.check()
        torch.cuda.synchronize()
        assert torch.equal(y[2], y[0]) and torch.equal(y[3], y[1])
    assert not torch.equal(y[0], y[1])
    sim.close()
