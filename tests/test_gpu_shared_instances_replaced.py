"""Batches of the fitting layer's instances (a base tensor with row scales)
whose tensors are replaced: plates of more than 64 modes, held dense, take a
new tensor in a context of any size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


def test_tensors_of_large_plates_can_be_replaced():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import fit, modal
    setup = fit.PlateSetup(n_t=70, n_in=40)
    rng = np.random.default_rng(2)
    th = np.array([6.0, 2.0, 0.8, 1.0, 5e-4])
    base = fit.plate_instance_shared(setup, th)
    insts = [dict(base, h_row_scale=base["h_row_scale"] * rng.uniform(0.5, 1.5)) for _ in range(100)]  # 78 MB
    batch, insts_b = modal.Sim(insts, FS), fit.plate_instances_shared(setup, np.stack([th] * 3))[0]
    assert batch.launches()["kernel"] == "streaming" and "mode_class" not in insts_b[0]
    H = rng.normal(size=base["Ht"].shape)
    H = (np.abs(base["Ht"]).max() * np.abs(base["h_row_scale"]).max() * 0.01 * (H + H.transpose(0, 2, 1))).astype(np.float32)
    batch.set_tensor(3, H)
    y = batch.run(60).cpu().numpy()
    lone = {k: v for k, v in base.items() if k not in ("h_row_scale", "mode_class")}
    ref = modal.Sim([dict(lone, Ht=H)], FS).run(60).cpu().numpy()[0]
    other = modal.Sim([insts[4]], FS).run(60).cpu().numpy()[0]
    assert np.linalg.norm(y[3] - ref) <= 1e-5 * np.linalg.norm(ref) and np.linalg.norm(ref) > 0
    assert np.linalg.norm(y[4] - other) <= 1e-5 * np.linalg.norm(other)
