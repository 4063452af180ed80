"""The modal state is stepped in FP64 on every path: after a run without a
force, the state equals the two-step recursion taken in numpy FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2505_05940_amd import modal
    return modal


# one-wave kernel; on-chip with a zero tensor; streaming, one and several
# slabs; streaming non-resident; shared tensor
CASES = [("linear", 3, 1, {}), ("linear", 200, 2, {}), ("vk", 5, 1, {}), ("vk", 70, 1, {}),
         ("vk", 9, 1, dict(waves=1, max_workgroups=3)), ("vk", 17, 32, {})]


@pytest.mark.parametrize("kind,n,batch,kw", CASES)
def test_state_is_fp64(gpu, kind, n, batch, kw):
    rng = np.random.default_rng(n)
    fs, steps, T = 44100.0, 4000, 1 / 44100.0
    H = np.zeros((3, n, n), np.float32)
    insts, ref = [], []
    for b in range(batch):
        w, g = 2 * np.pi * rng.uniform(50, 8000, n), rng.uniform(0.5, 20, n)
        x0 = rng.normal(size=n)
        inst = dict(kind=kind, omega=w, gamma=g, x0=x0, xm1=x0 * 0.9, c=rng.normal(size=n))
        if kind == "vk":
            inst["Ht"] = H
        insts.append(inst)
        r = T * T / (1 + g * T)
        m, p = -r * w * w, -(1 - g * T) / (1 + g * T)
        x, d = x0.copy(), x0 - inst["xm1"]
        for _ in range(steps):
            d = m * x - p * d
            x = x + d
        ref.append(x)
    sim = gpu.Sim(insts, fs, flags=gpu.FLAG_RECURSE, **kw)
    sim.run(steps)
    x, _ = sim.state()
    ref = np.concatenate(ref)
    # every step rounds X and d to half an ulp on both sides, each error
    # carried on by the damped oscillation at most |1 / sin(wT)| times the
    # relative size of d (about wT): 4 roundings a step, 2 sides
    tol = 8 * steps * 2.0 ** -53 * np.pi / 2
    assert np.max(np.abs(x - ref)) <= tol * np.max(np.abs(ref)) * 2
