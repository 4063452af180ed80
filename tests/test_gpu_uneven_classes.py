"""Tensors stored by class whose classes are of very unequal size (more than 64
modes paired with at most 12): every stored row of a transposed pair counts,
against the same tensor held dense.  FP32 sums over at most 100 products in
another order, 40 steps: 1e-5 of the output."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


@pytest.mark.parametrize("sizes", [(100, 8, 0, 0), (70, 3, 9, 40), (5, 130, 12, 66), (64, 4, 4, 64), (260, 2, 1, 7)])
@pytest.mark.parametrize("waves", [1, 4])
def test_unequal_classes(sizes, waves):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(sum(sizes))
    cls = rng.permutation(np.repeat(np.arange(4), sizes)).astype(np.uint8)
    n, nin = len(cls), 6
    H = rng.normal(size=(nin, n, n))
    H = H + H.transpose(0, 2, 1)
    for i in range(nin):  # one column class to each class: i xor 1, 2, 3 in turn, and i itself
        H[i] *= (cls[:, None] ^ cls[None, :]) == (1, 2, 3, 0)[i % 4]
    x0 = rng.normal(size=n) / np.sqrt(n)
    plate = dict(kind="vk", omega=2 * np.pi * np.sort(rng.uniform(80, 7000, n)), gamma=np.full(n, 4.0), x0=x0, xm1=x0,
                 c=rng.normal(size=n), Ht=(3e2 * H).astype(np.float32), mode_class=cls)
    y, moved = {}, None
    for flag in (0, modal.FLAG_NO_BLOCK):
        sim = modal.Sim([plate], FS, flags=flag, waves=waves, max_workgroups=2)
        assert sim.info()["blocked_instances"] == (flag == 0)
        y[flag] = sim.run(40).cpu().numpy()[0]
        sim.close()
    free = modal.Sim([dict(plate, Ht=np.zeros_like(plate["Ht"]))], FS)
    moved = np.linalg.norm(free.run(40).cpu().numpy()[0] - y[modal.FLAG_NO_BLOCK])
    free.close()
    a, b = y.values()
    assert np.isfinite(b).all() and moved > 1e-3 * np.linalg.norm(b)  # (the tensor matters)
    assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b)
