"""Runs of a context while another stream of the process is under capture: the
second run of a context, which takes pinned memory for its flags, and those
beside it, must neither fail nor end the capture, and give the outputs of the
same runs without one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


@pytest.mark.parametrize("mode", ["global", "thread_local"])
@pytest.mark.parametrize("kind", ["tension", "vk"])
def test_second_run_beside_a_capture(kind, mode):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    n = 20
    H = np.random.default_rng(1).normal(size=(8, n, n))
    inst = dict(kind=kind, omega=2 * np.pi * np.linspace(80, 5000, n), gamma=np.full(n, 5.0), x0=np.full(n, 1e-3),
                xm1=np.full(n, 1e-3), c=np.ones(n))
    if kind == "vk":
        inst["Ht"] = (3e4 * (H + H.transpose(0, 2, 1))).astype(np.float32)
    else:
        inst["lam"], inst["kappa"] = np.arange(1.0, n + 1), 1e6
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    sim = modal.Sim([inst], FS, flags=modal.FLAG_ASYNC, stream=side)
    whole = torch.empty((1, 300), device="cuda")
    sim.run(300, out=whole)
    sim.check()
    sim.close()
    sim = modal.Sim([inst], FS, flags=modal.FLAG_ASYNC, stream=side)
    y = [torch.empty((1, 100), device="cuda") for _ in range(3)]
    v = torch.arange(64.0, device="cuda")
    torch.cuda.synchronize()
    sim.run(100, out=y[0])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=other, capture_error_mode=mode):
        v.mul_(2.0)
        sim.run(100, out=y[1])
        sim.run(100, out=y[2])
    graph.replay()
    sim.check()
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(y, 1), whole)
    assert torch.equal(v.cpu(), 2.0 * torch.arange(64.0))
    sim.close()
