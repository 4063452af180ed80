"""The autotuner against the plans that modal_init chooses by itself: batches
that have a kernel of their own keep it when they are tuned, and a cache
written when they had none does not take it away."""
import ctypes as C
import json

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0


def _strings(n):
    k = np.arange(1.0, 13.0)
    return [dict(kind="tension", omega=2 * np.pi * 100 * k * (1 + 0.01 * b / n), gamma=np.full(12, 3.0),
                 x0=1e-3 / k, xm1=1e-3 / k, c=np.ones(12), lam=k ** 2, kappa=1e4) for b in range(n)]


def _plates(n, nt, nin):
    rng = np.random.default_rng(nt)
    H = rng.normal(size=(nin, nt, nt))
    H = (1e3 * (H + H.transpose(0, 2, 1))).astype(np.float32)
    return [dict(kind="vk", omega=2 * np.pi * np.linspace(80, 7000, nt), gamma=np.full(nt, 3.0), x0=np.full(nt, 1e-3),
                 xm1=np.full(nt, 1e-3), c=np.ones(nt), Ht=H.copy()) for _ in range(n)]


@pytest.mark.parametrize("name", ["strings", "small plates", "large plate"])
def test_tuned_batches_keep_their_kernel(tmp_path, name):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal, tune
    insts = dict(zip(["strings", "small plates", "large plate"],
                     [_strings(600), _plates(300, 24, 24), _plates(1, 100, 100)]))[name]
    cache = str(tmp_path / "tune.json")
    best = tune.autotune(insts, FS, shapes=((4, 2), (8, 1)), samples=100, cache=cache, split_costs=(32,))
    assert best == (0, 0, 0)
    assert tune.autotune(insts, FS, cache=cache) == best
    tuned, default = modal.Sim(insts, FS, tune_cache=cache), modal.Sim(insts, FS)
    assert tuned.info() == default.info()
    assert np.array_equal(tuned.run(200).cpu().numpy(), default.run(200).cpu().numpy())
    tuned.close()
    default.close()


def test_entries_of_the_first_set_of_plans_lapse(tmp_path):
    import torch
    from paper_2505_05940_amd import modal
    insts = _strings(300)

    class Props(C.Structure):  # the device's name opens hipDeviceProp_t
        _fields_ = [("name", C.c_char * 256), ("rest", C.c_char * 8192)]

    props = Props()
    assert modal.lib.hipGetDevicePropertiesR0600(C.byref(props), torch.cuda.current_device()) == 0
    h = 1469598103934665603
    data = props.name + np.array([len(insts), 0, 0] + [v for _ in insts for v in (1, 12, 0, 0, 0)], np.int32).tobytes()
    for byte in data:
        h = ((h ^ byte) * 1099511628211) % (1 << 64)
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({"%016x" % h: dict(waves=4, max_workgroups=256, split_cost_kb=0)}))
    sim = modal.Sim(insts, FS, tune_cache=str(cache))
    assert sim.info()["path"] == 3
    sim.close()
    cache.write_text(json.dumps({modal.tune_key(insts, FS): dict(waves=4, max_workgroups=256, split_cost_kb=0)}))
    sim = modal.Sim(insts, FS, tune_cache=str(cache))  # a current entry is taken
    assert sim.info()["path"] == 0
    sim.close()
