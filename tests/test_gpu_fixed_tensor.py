"""Tensors with mode classes in a batch of more plates than CUs are stored by
class and refused by set_tensor, on chip as where they stream; tensors without
classes, and any in a context that keeps them dense, can be replaced."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


@pytest.mark.parametrize("classed,flag,refused", [(True, "", True), (False, "", False), (True, "FLAG_NO_BLOCK", False),
                                                  (True, "FLAG_GRAD", False)])
def test_batches_larger_than_the_gpu(classed, flag, refused):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(1)
    n, batch = 12, torch.cuda.get_device_properties(0).multi_processor_count + 9
    cls = (np.arange(n) % 4).astype(np.uint8)

    def tensor():
        H = rng.normal(size=(5, n, n))
        H = 1e5 * (H + H.transpose(0, 2, 1))
        return (H * ((cls[:, None] ^ cls[None, :]) == 1)).astype(np.float32)

    x0 = 1e-3 * rng.normal(size=n)
    insts = [dict(kind="vk", omega=2 * np.pi * np.linspace(80, 7000, n), gamma=np.full(n, 4.0), x0=x0, xm1=x0,
                  c=rng.normal(size=n), Ht=tensor(), **(dict(mode_class=cls) if classed else {})) for _ in range(batch)]
    sim = modal.Sim(insts, FS, flags=getattr(modal, flag) if flag else 0)
    assert sim.launches()["kernel"] == "on-chip"
    H = tensor()
    if refused:
        with pytest.raises(modal.ModalError) as e:
            sim.set_tensor(7, H)
        assert e.value.status == "ESTATE"
        H = insts[7]["Ht"]
    else:
        sim.set_tensor(7, H)
    y = sim.run(90).cpu().numpy()[7]
    lone = {k: v for k, v in insts[7].items() if k != "mode_class"}
    ref = modal.Sim([dict(lone, Ht=H)], FS, waves=4, max_workgroups=4).run(90).cpu().numpy()[0]
    assert np.linalg.norm(y - ref) <= 1e-5 * np.linalg.norm(ref)
    sim.close()
