"""Batches whose instances the planner cuts although they are small (from half
a megabyte of tensor): each plate's output against the same plate alone, whose
route is another (relative 1e-5, the bar of the FP32 forces)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("modes,batch", [((100,), 20), ((66, 90, 130), 40)])
def test_split_small_instances(modes, batch):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal, physics
    insts = [physics.plate_instance(W.plate_vk(seed=70 + i, n_t=modes[i % len(modes)], family="sine", grid=None,
                                               n_steps=200)) for i in range(batch)]
    sim = modal.Sim(insts, 44100.0)
    info = sim.info()
    assert info["split_instances"] > 0 and info["blocked_instances"] == batch, info
    y = sim.run(200).double().cpu().numpy()
    sim.close()
    for i in (0, 1, batch - 1):
        one = modal.Sim([insts[i]], 44100.0)
        z = one.run(200).double().cpu().numpy()[0]
        one.close()
        assert np.linalg.norm(y[i] - z) < 1e-5 * np.linalg.norm(z), i
