"""Gradients with a tangent tensor of plates that step on chip: the trajectory
and the checkpoints that the on-chip kernel records are read back by the
streaming reverse sweep in groups of four modes, zeros past the last mode
included.  Mode counts on and off multiples of four, tensors held whole and by
mode class, a tension instance beside them, records and checkpoints reused and
made by the gradient call, in device memory that held NaNs before; against the
same gradients on an explicit launch shape (streaming kernels throughout).

Both sweeps are FP32 forces on an FP64 state, so they differ by about 1e-6 of
a gradient; a NaN or a neighbour's value in a pad is far outside 1e-4."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


def _nan_memory(modal):
    """Device memory of the sizes that a context allocates, full of NaNs, given back."""
    ptrs = []
    for size in (1 << 12, 1 << 14, 1 << 16, 1 << 18, 1 << 20):
        for _ in range(24):
            p = C.c_void_p()
            assert modal.lib.hipMalloc(C.byref(p), C.c_size_t(size)) == 0
            assert modal.lib.hipMemset(p, 0xFF, C.c_size_t(size)) == 0
            ptrs.append(p)
    assert modal.lib.hipDeviceSynchronize() == 0
    for p in ptrs:
        assert modal.lib.hipFree(p) == 0


def _plate(rng, n, n_in, classed):
    om = 2 * np.pi * np.sort(rng.uniform(80, 7000, n))
    H = rng.normal(size=(n_in, n, n))
    H = 0.5 * (H + H.transpose(0, 2, 1)) * np.sqrt(4.0 / (n * n_in))
    inst = dict(kind="vk", omega=om, gamma=rng.uniform(1, 30, n), x0=1e-3 * rng.normal(size=n), c=rng.normal(size=n))
    if classed:
        cls = rng.integers(4, size=n)
        for i in range(n_in):
            H[i] *= (cls[:, None] ^ cls[None, :]) == rng.integers(4)
        inst["mode_class"] = cls.astype(np.uint8)
    inst["Ht"] = (H * 3e6).astype(np.float32)
    inst["xm1"] = inst["x0"].copy()
    return inst


@pytest.mark.parametrize("classed", [False, True])
@pytest.mark.parametrize("runs", [(), (200,), (90, 110)])
@pytest.mark.parametrize("n", [1, 14, 37, 40, 63])
def test_tangent_of_plates_on_chip(n, runs, classed):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(n)
    n_in = min(n + 2, 24)
    insts = [_plate(rng, n, n_in, classed),
             dict(kind="tension", omega=2 * np.pi * np.arange(1, 8) * 150.0, gamma=np.full(7, 3.0),
                  x0=1e-3 * rng.normal(size=7), xm1=np.zeros(7), c=rng.normal(size=7), lam=np.arange(1, 8) ** 2.0,
                  kappa=1e4)]
    Hd = 0.1 * insts[0]["Ht"]
    g = torch.tensor(1e3 * rng.normal(size=(2, 200)), dtype=torch.float32, device="cuda")
    got = []
    for kw in ({}, dict(waves=4, max_workgroups=32)):
        _nan_memory(modal)
        sim = modal.Sim(insts, FS, flags=modal.FLAG_GRAD, **kw)
        sim.set_tangent(0, Hd)
        for k in runs:
            sim.run(k)
        got.append(sim.grad(200, g))
        sim.close()
    for key in got[0]:
        x, y = (np.concatenate([np.ravel(a) for a in r[key]]) for r in got)
        assert np.isfinite(x).all(), key
        assert np.linalg.norm(x - y) <= 1e-4 * np.linalg.norm(y), key
