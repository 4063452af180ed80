"""A batch of small plates whose tensors fit the GPU's free memory stored by
class but not dense: it streams its blocks, as it does where memory is plenty
only when asked to, and gives the outputs of the on-chip kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, NT, BATCH = 44100.0, 40, 9000


def test_small_plates_in_little_memory():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(1)
    cls = (np.arange(NT) % 4).astype(np.uint8)
    H = rng.normal(size=(NT, NT, NT)).astype(np.float32)
    H = (H + H.transpose(0, 2, 1)) * np.float32(1e4)
    for n in range(NT):
        H[n] *= (cls[:, None] ^ cls[None, :]) == n % 4
    x0 = 1e-3 * rng.normal(size=NT)
    plate = dict(kind="vk", omega=2 * np.pi * np.linspace(80, 7000, NT), gamma=np.full(NT, 4.0), x0=x0, xm1=x0,
                 c=rng.normal(size=NT), Ht=H, mode_class=cls)
    few = modal.Sim([plate], FS, flags=modal.FLAG_NO_SHARED)
    assert few.info()["path"] == 3
    ref = few.run(100).cpu().numpy()[0]
    few.close()
    # 2.3 GB dense, 0.4 GB by class; leave 2 GB
    torch.cuda.empty_cache()
    hog = torch.empty(torch.cuda.mem_get_info()[0] - (2 << 30), dtype=torch.uint8, device="cuda")
    try:
        sim = modal.Sim([plate] * BATCH, FS, flags=modal.FLAG_NO_SHARED)
        info = sim.info()
        assert info["path"] == 0 and info["blocked_instances"] == BATCH
        y = sim.run(100).cpu().numpy()
        sim.close()
    finally:
        del hog
        torch.cuda.empty_cache()
    assert np.isfinite(ref).all()
    for b in (0, 1, BATCH // 2, BATCH - 1):
        assert np.linalg.norm(y[b] - ref) < 1e-5 * np.linalg.norm(ref)
    sim = modal.Sim([plate] * BATCH, FS, flags=modal.FLAG_NO_SHARED)
    assert sim.info()["path"] == 3  # with room, on chip
    assert np.array_equal(sim.run(100).cpu().numpy()[BATCH - 1], ref)
    sim.close()
