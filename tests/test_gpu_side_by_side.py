"""Contexts whose workgroups wait for each other's forces, on several streams
at once: batches of plates in slabs that fill the GPU, lone plates on the
latency kernel that fit beside each other and that do not, gradients, graph
launches and calls from several threads.  All must end (a launch that is half
resident beside another half runs into the wait limit of 4 s and is reported)
with the bits of the same calls alone."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


def _plate(rng, nt, nin):
    H = rng.normal(size=(nin, nt, nt)).astype(np.float32)
    H = (H + H.transpose(0, 2, 1)) * np.float32(4e3 / np.sqrt(nt * nin))
    x0 = rng.normal(size=nt) / np.sqrt(nt)
    return dict(kind="vk", omega=2 * np.pi * np.sort(rng.uniform(50, 6000, nt)), gamma=rng.uniform(0.5, 20, nt), x0=x0,
                xm1=0.98 * x0, c=rng.normal(size=nt), Ht=H)


# name: (number of plates, modes, rows, steps)
BATCHES = {"slabs": (96, 90, 60, 600), "big": (1, 200, 200, 12000), "small": (1, 100, 100, 12000)}


@pytest.fixture(scope="module")
def plates():
    rng = np.random.default_rng(3)
    return {k: [_plate(rng, nt, nin) for _ in range(n)] for k, (n, nt, nin, _) in BATCHES.items()}


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("kinds", [("slabs", "slabs"), ("big", "big", "big"), ("slabs", "big", "small", "slabs"),
                                   ("small",) * 6])
def test_runs_on_several_streams(plates, kinds, graph):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    flags = modal.FLAG_ASYNC | (modal.FLAG_GRAPH if graph else 0)
    streams = [torch.cuda.Stream() for _ in kinds]
    sims = [modal.Sim(plates[k], FS, flags=flags, stream=s) for k, s in zip(kinds, streams)]
    assert all(s.info()["split_instances"] for s in sims)
    outs = [torch.empty((s.batch, BATCHES[k][3]), device="cuda") for k, s in zip(kinds, sims)]
    torch.cuda.synchronize()
    for _ in range(2):
        for s, y in zip(sims, outs):
            s.reset()
            s.run(y.shape[1], out=y)
    for s in sims:
        s.check()
    alone = {}
    for k, s, y in zip(kinds, sims, outs):
        if k not in alone:
            s.reset()
            alone[k] = y.clone()
            torch.cuda.synchronize()
            s.run(y.shape[1], out=y)
            s.check()
            assert torch.equal(y, alone[k])
        assert torch.isfinite(y).all() and torch.equal(y, alone[k])
    for s in sims:
        s.close()


def test_calls_from_several_threads(plates):
    import torch
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(6)
    ybar = torch.tensor(rng.normal(size=(1, 2000)), dtype=torch.float32, device="cuda")
    kinds = ("big", "slabs", "big", "small", "slabs", "small")

    def call(kind, out, i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            grad = kind != "slabs"
            sim = modal.Sim(plates[kind], FS, flags=modal.FLAG_GRAD if grad else 0, stream=stream)
            res = []
            for _ in range(3):
                sim.reset()
                res.append(sim.run(400).cpu().numpy())
                if grad:
                    g = sim.grad(2000, ybar)
                    res.append(np.concatenate([g["omega"][0], g["row"][0], g["x0"][0]]))
            sim.close()
            out[i] = res

    torch.cuda.synchronize()
    alone = {}
    for k in set(kinds):
        call(k, alone, k)
    got = [None] * len(kinds)
    threads = [threading.Thread(target=call, args=(k, got, i)) for i, k in enumerate(kinds)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, r in zip(kinds, got):
        assert r is not None and len(r) == len(alone[k])
        assert all(np.isfinite(a).all() and np.array_equal(a, b) for a, b in zip(r, alone[k])), k
