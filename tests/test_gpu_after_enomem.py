"""A call that reports that memory has run out leaves no error behind: the next
call, of the same or another part of the library, succeeds."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_calls_after_a_failed_allocation():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    from paper_2505_05940_amd.mlp import MLP
    n = 16
    inst = dict(kind="tension", omega=np.linspace(500.0, 9000.0, n), gamma=np.full(n, 3.0), x0=np.full(n, 1e-3),
                xm1=np.full(n, 1e-3), c=np.ones(n), lam=np.ones(n), kappa=1e3)
    ptr = lambda a: a.ctypes.data_as(C.c_void_p)
    coef, w, H = np.array([[-1.2, 0.9, 0.3, -0.1, 2.0]]), np.linspace(0.1, 3.0, 9), np.zeros((9, 2))
    x = torch.randn(4, 3, device="cuda")
    sim, net = modal.Sim([inst], 44100.0), MLP([3, 2], max_batch=4)
    net.init_params(seed=1)
    ref, y_ref = sim.run(30).clone(), net.forward(x).clone()
    calls = [lambda: sim.run(30), lambda: net.forward(x), lambda: modal.Sim([inst], 44100.0).run(30),
             lambda: modal.lib.modal_tf_response(ptr(coef), ptr(np.array([0, 1], np.int32)), 1, ptr(w), 9, ptr(H), None)]
    for call in calls:
        sim.reset()
        off = np.zeros(65536, np.int32)
        code = modal.lib.modal_tf_response(ptr(coef), ptr(off), 65535, ptr(np.ones(1 << 20)), 1 << 20, ptr(H), None)
        assert modal.STATUS[code] == "ENOMEM"  # 1.1 TB of output
        got = call()
        if isinstance(got, int):
            assert got == 0, modal.lib.modal_last_error()
        else:
            assert torch.equal(got, ref if got.shape == ref.shape else y_ref)
    net.close()
    sim.close()
