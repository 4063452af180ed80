"""Launches of one step on the on-chip kernel, whose waves each step a copy of
an instance's state that one of them writes back: a batch of von Karman,
tension-modulated and linear instances in many short runs, and in chunks, must
give the bits of one long run, and a gradient made from recorded short runs
those of one made from a long one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS = 44100.0, 300


def _instances(rng):
    out = []
    for kind, n in [("vk", 12), ("tension", 30), ("linear", 64), ("tension", 3), ("vk", 33), ("linear", 5)] * 12:
        w = 2 * np.pi * np.sort(rng.uniform(80, 7000, n))
        p = dict(kind=kind, omega=w, gamma=rng.uniform(1, 30, n), x0=1e-3 * rng.normal(size=n), c=rng.normal(size=n))
        p["xm1"] = 0.99 * p["x0"]
        if kind == "vk":
            H = rng.normal(size=(9, n, n))
            p["Ht"] = (3e6 * (H + H.transpose(0, 2, 1)) / n).astype(np.float32)
        if kind == "tension":
            p["lam"], p["kappa"] = np.arange(1.0, n + 1), 1e6
        if n % 2:
            p["b_ext"], p["e_ext"] = rng.normal(size=n), rng.normal(size=70).astype(np.float32)
        out.append(p)
    return out


def test_one_step_runs_equal_a_long_one():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    insts = _instances(np.random.default_rng(4))
    sim = modal.Sim(insts, FS)
    assert sim.info()["path"] == 3
    whole = sim.run(STEPS).cpu().numpy()
    state = sim.state()
    assert np.isfinite(whole).all()
    sim.reset()
    parts = [sim.run(k).cpu().numpy() for k in [1] * 200 + [2] * 30 + [5] * 8]
    assert np.array_equal(np.concatenate(parts, 1), whole)
    assert all(np.array_equal(a, b) for a, b in zip(sim.state(), state))
    sim.close()
    sim = modal.Sim(insts, FS, chunk_steps=1)
    assert np.array_equal(sim.run(STEPS).cpu().numpy(), whole)
    sim.close()


def test_gradients_of_one_step_runs():
    import torch
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(5)
    insts = _instances(rng)
    g = torch.tensor(rng.normal(size=(len(insts), STEPS)), dtype=torch.float32, device="cuda")
    got = []
    for chunk in (0, 1):
        sim = modal.Sim(insts, FS, flags=modal.FLAG_GRAD, chunk_steps=chunk)
        sim.run(STEPS)
        got.append(sim.grad(STEPS, g))
        sim.close()
    for key in got[0]:
        assert all(np.array_equal(a, b) for a, b in zip(got[0][key], got[1][key])), key
