"""Launches of one step on the latency kernel, whose slabs all start from the
state that one of them writes back: lone plates in slabs with rows for few of
their waves and for all, exchanging directly and through the slabs that own
modes, in many short runs, must give the bits of one long run."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS = 44100.0, 240


@pytest.mark.parametrize("nt,nin", [(65, 9), (100, 100), (131, 129), (257, 40)])
def test_one_step_runs_equal_a_long_one(nt, nin):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(nt)
    H = rng.normal(size=(nin, nt, nt))
    H = (H + H.transpose(0, 2, 1)) * (4e3 / np.sqrt(nt * nin))
    x0 = rng.normal(size=nt) / np.sqrt(nt)
    plate = dict(kind="vk", omega=2 * np.pi * np.sort(rng.uniform(50, 6000, nt)), gamma=rng.uniform(0.5, 20, nt), x0=x0,
                 xm1=0.98 * x0, c=rng.normal(size=nt), Ht=H.astype(np.float32))
    sim = modal.Sim([plate], FS)
    whole = sim.run(STEPS).cpu().numpy()
    state = sim.state()
    assert np.isfinite(whole).all()
    sim.reset()
    parts = [sim.run(k).cpu().numpy() for k in [1] * 200 + [2] * 20]
    assert np.array_equal(np.concatenate(parts, 1), whole)
    assert all(np.array_equal(a, b) for a, b in zip(sim.state(), state))
    sim.close()
