"""The wave kernels (batches without a coupling tensor): every lanes-per-instance
and modes-per-lane shape, full and partly filled waves, driven and free, against
the FP64 recursion and the oracle's reverse pass.  Bars as for the other
kernels: 1e-5 relative L2 per output signal, 1e-4 per gradient vector."""
import numpy as np
import pytest

from oracle import adjoint as OA

pytestmark = pytest.mark.gpu
FS = 44100.0


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    from paper_2505_05940_amd import modal
    return modal, torch


def _instance(rng, n, kind, n_exc):
    k = np.arange(1, n + 1)
    om = 2 * np.pi * np.sort(rng.uniform(60, 9000, n))
    inst = dict(kind=kind, omega=om, gamma=rng.uniform(0.5, 30, n), x0=1e-3 * rng.normal(size=n) / k,
                xm1=1e-3 * rng.normal(size=n) / k, c=rng.normal(size=n))
    inst["xm1"] = inst["x0"] + 0.02 * (inst["xm1"] - inst["x0"])
    if kind == "tension":
        inst["lam"] = (k * np.pi / 0.65) ** 2
        inst["kappa"] = 2e7 / n
    if n_exc:
        inst["b_ext"] = 20 * rng.normal(size=n)
        inst["e_ext"] = rng.normal(size=n_exc).astype(np.float32)
    return inst


def _run64(inst, steps):
    T = 1 / FS
    om, ga = inst["omega"], inst["gamma"]
    r = T * T / (1 + ga * T)
    x, d = inst["x0"].copy(), inst["x0"] - inst["xm1"]
    y = np.empty(steps)
    for s in range(steps):
        y[s] = inst["c"] @ x
        f = 0.0
        if inst["kind"] == "tension":
            f = inst["kappa"] * inst["lam"] * x * np.sum(inst["lam"] * x * x)
        if inst.get("e_ext") is not None and s < len(inst["e_ext"]):
            f = f - inst["b_ext"] * float(inst["e_ext"][s])
        d = -r * om * om * x + (1 - ga * T) / (1 + ga * T) * d - r * f
        x = x + d
    return y


# (modes, batch): one and several modes per lane on 16, 32 and 64 lanes; the
# large batches take fewer lanes and leave the last wave partly filled
@pytest.mark.parametrize("n,batch", [(1, 1), (16, 3), (17, 1), (32, 5), (33, 1), (64, 2), (65, 1), (256, 1),
                                     (30, 2050), (60, 4099), (100, 1027)])
def test_wave_run(gpu, n, batch):
    modal, torch = gpu
    rng = np.random.default_rng(n)
    kinds = ["tension", "linear"] if n != 65 else ["linear"]
    base = [_instance(rng, n if i % 3 else max(1, n - 1), kinds[i % len(kinds)], (0, 90)[i % 2]) for i in range(5)]
    insts = [base[b % 5] for b in range(batch)]
    steps = 200  # not a multiple of a chunk
    sim = modal.Sim(insts, FS, flags=modal.FLAG_RECURSE)
    assert sim.info()["path"] == 3
    a, b = sim.run(77), sim.run(steps - 77)
    y = torch.cat([a, b], 1).double().cpu().numpy()
    for i in {0, 1, 2, 3, 4, batch - 1}:
        if i < batch:
            ref = _run64(insts[i], steps)
            assert np.linalg.norm(y[i] - ref) <= 1e-5 * np.linalg.norm(ref), i
    assert all(np.array_equal(y[b], y[b % 5]) for b in range(batch))


@pytest.mark.parametrize("n,batch,ckpt", [(1, 1, 0), (12, 1, 0), (16, 2, 100), (20, 3, 0), (33, 1, 0), (100, 1, 64),
                                          (200, 2, 0), (60, 1100, 0)])
def test_wave_grad(gpu, n, batch, ckpt):
    modal, torch = gpu
    rng = np.random.default_rng(100 + n)
    base = [_instance(rng, n if i != 1 else max(1, n - 1), "tension" if n > 1 else "linear", 0) for i in range(2)]
    insts = [base[b % 2] for b in range(batch)]
    steps = 203
    g = rng.normal(size=(2, steps)).astype(np.float32)
    gy = torch.tensor(g, device="cuda")[torch.arange(batch, device="cuda") % 2].contiguous()
    sim = modal.Sim(insts, FS, flags=modal.FLAG_GRAD)
    if batch == 3:
        sim.run(steps)  # the gradient then reuses the run's record
    res = sim.grad(steps, gy, ckpt_every=ckpt)
    for i in {0, 1, batch - 1}:
        if i >= batch:
            continue
        inst = dict(insts[i])
        r = OA.reverse(inst, steps, FS, g[i % 2].astype(float))
        om, ga = OA.sv_omega_gamma_grads(r, inst["omega"], inst["gamma"], 1 / FS)
        ref = dict(omega=om, gamma=ga, c=r["c"], x0=r["x0"], xm1=r["xm1"])
        for k, v in ref.items():
            assert np.linalg.norm(res[k][i] - v) <= 1e-4 * np.linalg.norm(v), (i, k)
        if inst["kind"] == "tension":
            assert abs(res["scale"][i] - r["scale"]) <= 1e-4 * abs(r["scale"]), i
