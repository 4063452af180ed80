"""Launches that a caller captured before a tensor was replaced: their replays
go on with the new tensor, for tensors of the classes given at the start and,
in contexts that keep tensors dense, for any; where the captured launches hold
the tensor by class and the new one has other entries, set_tensor says so and
changes nothing."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS = 44100.0, 80


def _tensor(rng, n, n_in, cls=None):
    H = rng.normal(size=(n_in, n, n))
    H = 0.5 * (H + H.transpose(0, 2, 1)) * np.sqrt(4.0 / (n * n_in))
    if cls is not None:
        for i in range(n_in):
            H[i] *= (cls[:, None] ^ cls[None, :]) == i % 4
    return (3e6 * H).astype(np.float32)


def _plate(rng, n, n_in, cls):
    x0 = 1e-3 * rng.normal(size=n)
    return dict(kind="vk", omega=2 * np.pi * np.sort(rng.uniform(80, 7000, n)), gamma=rng.uniform(1, 30, n), x0=x0,
                xm1=x0.copy(), c=rng.normal(size=n), Ht=_tensor(rng, n, n_in, cls), mode_class=cls.astype(np.uint8))


# tensors that fit one workgroup whole, and one that does only by class
@pytest.mark.parametrize("n,n_in", [(18, 12), (40, 40), (56, 56)])
@pytest.mark.parametrize("flags", ["", "grad", "dense"])
@pytest.mark.parametrize("noalloc", [False, True])
def test_replays_after_a_replaced_tensor(n, n_in, flags, noalloc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    fl = modal.FLAG_ASYNC | {"": 0, "grad": modal.FLAG_GRAD, "dense": modal.FLAG_NO_BLOCK}[flags]
    rng = np.random.default_rng(n)
    cls = np.arange(n) % 4
    p = _plate(rng, n, n_in, cls)
    stream = torch.cuda.Stream()
    sim = modal.Sim([p], FS, flags=fl, stream=stream)
    y = torch.empty((1, STEPS), device="cuda")
    torch.cuda.synchronize()
    step = sim.run_noalloc if noalloc else sim.run
    step(STEPS, out=y)
    sim.check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        step(STEPS, out=y)
    for H, any_kind in [(_tensor(rng, n, n_in, cls), False), (_tensor(rng, n, n_in), True), (_tensor(rng, n, n_in), True)]:
        dev = torch.tensor(H, device="cuda")
        torch.cuda.synchronize()
        if any_kind and not flags:
            before = p["Ht"]
            with pytest.raises(modal.ModalError) as e:
                sim.set_tensor(0, dev)
            assert e.value.status == "ESTATE"
        else:
            sim.set_tensor(0, dev)
            before = H
        p = dict(p, Ht=before)
        fresh = modal.Sim([{k: v for k, v in p.items() if k != "mode_class"}], FS, waves=4, max_workgroups=8)
        ref = fresh.run(2 * STEPS).cpu().numpy()[0]
        fresh.close()
        sim.reset()
        torch.cuda.synchronize()
        for part in range(2):
            graph.replay()
            torch.cuda.synchronize()
            got = y.cpu().numpy()[0]
            want = ref[part * STEPS:(part + 1) * STEPS]
            assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), (any_kind, part)
        sim.check()
    sim.close()
