"""Transfer-function calls at the ends of their ranges: a bound on the modes of
an instance far above what there is, more frequencies than one launch takes
(2^27), and a gradient that the GPU's memory cannot hold.  The response of one mode is a closed form in numpy; the device's
float-float arithmetic keeps about 48 bits of it."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
COEF = np.array([[-1.2, 0.9, 0.3, -0.1, 2.0], [0.4, 0.5, 1.0, 0.2, 0.7], [-0.3, 0.81, 0.1, 0.6, 1.1]])


def _h(w, coef):
    z = np.exp(1j * w)
    return sum(c[4] * (c[2] * z + c[3]) / (z * z + c[0] * z + c[1]) for c in coef)


def _ptr(a):
    return a.ctypes.data_as(C.c_void_p)


def _check(modal, code):
    assert code == 0, modal.lib.modal_last_error()


@pytest.mark.parametrize("max_modes", [2, 3, 1 << 24, (1 << 31) - 1])
def test_bound_on_the_modes(max_modes):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    off = np.array([0, 2, 3], np.int32)
    w = np.linspace(0.1, 3.0, 37)
    g = np.random.default_rng(1).normal(size=(2, 37, 2))
    out = np.zeros((3, 5))
    _check(modal, modal.lib.modal_tf_grad(_ptr(COEF), _ptr(off), 2, max_modes, _ptr(w), 37, _ptr(g), _ptr(out), None))
    for m in range(3):
        b = 0 if m < 2 else 1
        for i in range(5):
            d = COEF[m:m + 1].repeat(2, 0)
            d[0, i] += 1e-6
            d[1, i] -= 1e-6
            diff = (_h(w, d[:1]) - _h(w, d[1:])) / 2e-6
            ref = np.sum(g[b, :, 0] * diff.real + g[b, :, 1] * diff.imag)
            assert abs(out[m, i] - ref) <= 1e-7 * np.sum(np.abs(g[b]) * np.abs(diff)[:, None])


def test_more_frequencies_than_a_launch_takes():
    import torch
    from paper_2505_05940_amd import modal
    n = (1 << 28) + 21
    off = np.array([0, 1], np.int32)
    w = np.full(n, 1.0)
    at = np.array([0, 1, 15, 16, (1 << 27) - 1, 1 << 27, (1 << 27) + 17, (1 << 28) - 1, 1 << 28, n - 2, n - 1])
    w[at] = np.linspace(0.2, 2.9, len(at))
    H = np.empty((n, 2))
    _check(modal, modal.lib.modal_tf_response(_ptr(COEF[:1].copy()), _ptr(off), 1, _ptr(w), n, _ptr(H), None))
    ref = _h(w[at], COEF[:1])
    assert np.allclose(H[at, 0] + 1j * H[at, 1], ref, rtol=1e-11, atol=0)
    base = _h(np.ones(1), COEF[:1])[0]
    rest = np.random.default_rng(2).integers(0, n, 100000)
    rest = rest[~np.isin(rest, at)]
    assert np.allclose(H[rest, 0], base.real, rtol=1e-11, atol=0) and np.allclose(H[rest, 1], base.imag, rtol=1e-11, atol=0)


def test_gradient_beyond_the_memory():
    """1.1 TB of dL/dH: refused before the host copies any of it (so the array
    given for it need not exist)."""
    import torch
    from paper_2505_05940_amd import modal
    n, batch = 1 << 20, 65535
    off = np.zeros(batch + 1, np.int32)
    off[1:] = 1
    w, out = np.full(n, 1.0), np.zeros((1, 5))
    code = modal.lib.modal_tf_grad(_ptr(COEF[:1].copy()), _ptr(off), batch, 1, _ptr(w), n, _ptr(np.zeros(2)), _ptr(out), None)
    assert modal.STATUS[code] == "ENOMEM"
