"""The step counter, kept by the host for eager launches and by the device for
captured ones: eager runs, replays of a captured run and a reset in turn give
the samples of one uninterrupted run (the excitation makes every step's index
count), on each path that steps a state."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    from paper_2505_05940_amd import modal
    return modal, torch


def _instances(path):
    rng = np.random.default_rng(len(path))
    n, batch = {"wave": (12, 3), "chip": (9, 2), "stream": (70, 1), "slabs": (70, 1)}[path]
    H = rng.normal(size=(20, n, n)).astype(np.float32)
    H = 1e4 * (H + H.transpose(0, 2, 1))
    out = []
    for _ in range(batch):
        x0 = 1e-3 * rng.normal(size=n)
        inst = dict(kind="vk" if path != "wave" else "linear", omega=2 * np.pi * rng.uniform(80, 6000, n),
                    gamma=rng.uniform(1, 20, n), x0=x0, xm1=x0.copy(), c=rng.normal(size=n),
                    b_ext=100 * rng.normal(size=n), e_ext=rng.normal(size=900).astype(np.float32))
        if path != "wave":
            inst["Ht"] = H
        out.append(inst)
    return out


@pytest.mark.parametrize("path", ["wave", "chip", "stream", "slabs"])
def test_eager_and_captured_runs_share_the_counter(gpu, path):
    modal, torch = gpu
    insts = _instances(path)
    kw = dict(waves=8, max_workgroups=1) if path == "stream" else {}
    flags = modal.FLAG_RECURSE | modal.FLAG_NO_SHARED
    whole = modal.Sim(insts, FS, flags=flags, **kw).run(700).cpu().numpy()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = modal.Sim(insts, FS, flags=flags | modal.FLAG_ASYNC, stream=stream, **kw)
        out = torch.zeros(len(insts), 100, device="cuda")
        for _ in range(2):
            got = [sim.run(150).cpu().numpy()]
            sim.run_noalloc(100, out)
            got.append(out.cpu().numpy())
            stream.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                sim.run_noalloc(100, out)
            for _ in range(3):
                g.replay()
                stream.synchronize()
                got.append(out.cpu().numpy())
            got.append(sim.run(150).cpu().numpy())
            sim.check()
            assert np.array_equal(np.concatenate(got, 1), whole)
            sim.reset()
