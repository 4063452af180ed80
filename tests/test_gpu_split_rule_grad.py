"""Gradients of a batch of plates that only the lower bound on cut instances
cuts into slabs (72 modes, 1.2 MB of tensor each, 75 MB together), against the
same plates on a few workgroups: FP32 forces summed in another order, so 1e-5
(as for the latency kernel's gradients)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS, BATCH, NT, NIN = 44100.0, 100, 60, 72, 60


def test_gradients_of_cut_plates():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(7)
    H = rng.normal(size=(NIN, NT, NT))
    H = ((H + H.transpose(0, 2, 1)) * (4e3 / np.sqrt(NT * NIN))).astype(np.float32)
    plates = []
    for _ in range(BATCH):
        x0 = rng.normal(size=NT) / np.sqrt(NT)
        plates.append(dict(kind="vk", omega=2 * np.pi * np.sort(rng.uniform(50, 6000, NT)), gamma=rng.uniform(0.5, 20, NT),
                           x0=x0, xm1=0.98 * x0, c=rng.normal(size=NT), Ht=H, h_row_scale=rng.uniform(0.5, 1.5, NIN)))
    g = torch.tensor(rng.normal(size=(BATCH, STEPS)), dtype=torch.float32, device="cuda")
    got = []
    for kw in ({}, dict(waves=4, max_workgroups=8)):
        sim = modal.Sim(plates, FS, flags=modal.FLAG_GRAD, **kw)
        v, cut = sim.launches(), sim.info()["split_instances"]
        assert v["kernel"] == v["reverse"] == "streaming"
        assert (cut > BATCH // 2) == (not kw), cut
        y = sim.run(STEPS).cpu().numpy()
        res = sim.grad(STEPS, g)
        got.append([y] + [np.stack(res[k]) for k in ("omega", "gamma", "c", "x0", "xm1", "row")])
        sim.close()
    for a, b in zip(*got):
        for i in range(BATCH):
            assert np.linalg.norm(a[i] - b[i]) <= 1e-5 * np.linalg.norm(b[i])
