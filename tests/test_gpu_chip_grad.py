"""The on-chip kernels at the edges of their register tiles: tensors held whole
and by mode class, forward and reverse, one instance and more than there are
CUs, and replaced tensors, against the FP64 oracle's loop and reverse pass
(bars as for the streaming kernels: 1e-5 relative L2 per output signal, 1e-4
per gradient)."""
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


def rel(a, b):
    a, b = np.asarray(a, float), np.asarray(b, float)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def _plate(rng, n, n_in, classes=None, forced=False):
    """A random symmetric tensor, strong enough to matter; with `classes` (a
    size per class) only the entries between a class and its partner."""
    om = 2 * np.pi * np.sort(rng.uniform(80, 7000, n))
    H = rng.normal(size=(n_in, n, n))
    H = 0.5 * (H + H.transpose(0, 2, 1)) * np.sqrt(4.0 / (n * n_in))
    inst = dict(kind="vk", omega=om, gamma=rng.uniform(1, 30, n), x0=1e-3 * rng.normal(size=n), c=rng.normal(size=n))
    if classes is not None:
        cls = rng.permutation(np.repeat(np.arange(4), classes))
        for i in range(n_in):
            H[i] *= (cls[:, None] ^ cls[None, :]) == rng.integers(4)
        inst["mode_class"] = cls.astype(np.uint8)
    inst["Ht"] = (H * 3e6).astype(np.float32)
    inst["xm1"] = inst["x0"].copy()
    if forced:
        inst["b_ext"] = 20 * rng.normal(size=n)
        inst["e_ext"] = rng.normal(size=70).astype(np.float32)
    return inst


def _check(modal, torch, insts, steps, ckpt, pre, tensor=True):
    oracle = [dict(i, Ht=i["Ht"].astype(np.float64)) for i in insts]
    rng = np.random.default_rng(steps)
    g = (1e3 * rng.normal(size=(len(insts), steps))).astype(np.float32)
    sim = modal.Sim(insts, FS, flags=modal.FLAG_GRAD)
    run = modal.Sim(insts, FS, flags=modal.FLAG_NO_SHARED)
    assert run.info()["path"] == 3
    y = torch.cat([run.run(steps // 3), run.run(steps - steps // 3)], 1).double().cpu().numpy()
    if pre:
        yg = sim.run(steps)
        assert np.array_equal(yg.double().cpu().numpy(), y)
    res = sim.grad(steps, torch.tensor(g, device="cuda"), ckpt_every=ckpt, tensor=tensor)
    for b in sorted({0, 1, len(insts) - 1} & set(range(len(insts)))):
        ref_y = OA.forward(oracle[b], steps, FS)[0]
        assert rel(y[b], ref_y) < 1e-5, (b, rel(y[b], ref_y))
        r = OA.reverse(oracle[b], steps, FS, g[b].astype(float), full_tensor=tensor)
        om, ga = OA.sv_omega_gamma_grads(r, insts[b]["omega"], insts[b]["gamma"], 1 / FS)
        for k, v in dict(omega=om, gamma=ga, c=r["c"], x0=r["x0"], xm1=r["xm1"], row=r["row"],
                         scale=[r["scale"]]).items():
            got = [res[k][b]] if k == "scale" else res[k][b]
            assert rel(got, v) < 1e-4, (b, k, rel(got, v))
        if tensor:
            assert rel(res["H"][b].double().cpu().numpy(), r["H"]) < 1e-4, b


# whole tensors: one mode, the widest register tile, tiles whose reverse sweep
# keeps columns in LDS, few and many rows
@pytest.mark.parametrize("n,n_in", [(1, 1), (8, 8), (9, 17), (12, 96), (16, 90), (20, 75), (24, 64), (32, 48), (40, 40),
                                    (48, 32), (64, 24), (64, 2)])
def test_whole_tensor(gpu, n, n_in):
    modal, torch = gpu
    inst = _plate(np.random.default_rng(n * 100 + n_in), n, n_in, forced=n % 3 == 0)
    _check(modal, torch, [inst], 150, 0 if n % 2 else 64, n % 2 == 1)


# class sizes: one class, uneven ones, an empty one, tiles at their edges
@pytest.mark.parametrize("classes,n_in", [((3, 0, 0, 0), 5), ((13, 9, 10, 8), 40), ((16, 16, 16, 16), 60),
                                          ((17, 12, 11, 10), 50), ((1, 2, 3, 4), 33), ((20, 0, 21, 10), 40)])
def test_classes(gpu, classes, n_in):
    modal, torch = gpu
    inst = _plate(np.random.default_rng(sum(classes) + n_in), sum(classes), n_in, classes)
    _check(modal, torch, [inst, _plate(np.random.default_rng(1), 7, 3)], 145, 0, True)


def test_more_instances_than_cus(gpu):
    modal, torch = gpu
    rng = np.random.default_rng(3)
    base = [_plate(rng, 10, 11, (3, 3, 2, 2)), _plate(rng, 6, 4)]
    _check(modal, torch, [base[b % 2] for b in range(521)], 40, 0, True, tensor=False)


@pytest.mark.parametrize("classes,n_in,grad", [((4, 3, 3, 2), 12, False), ((4, 3, 3, 2), 12, True),
                                               ((16, 14, 14, 12), 56, False), ((16, 14, 14, 12), 56, True)])
def test_replaced_tensor_is_held_whole(gpu, classes, n_in, grad):
    """A tensor with entries that the first one's classes ruled out, set mid-run:
    small enough to be held whole, and too large for it."""
    modal, torch = gpu
    rng = np.random.default_rng(8)
    n = sum(classes)
    a, b = _plate(rng, n, n_in, classes), _plate(rng, n, n_in)
    sim = modal.Sim([a], FS, flags=modal.FLAG_GRAD if grad else 0)
    sim.run(50)
    sim.set_tensor(0, b["Ht"])
    y = sim.run(60)[0].double().cpu().numpy()
    # the oracle: 50 steps of the first plate, then the second from that state
    _, X, d, _ = OA.forward(dict(a, Ht=a["Ht"].astype(float)), 51, FS)
    ref = OA.forward(dict(a, Ht=b["Ht"].astype(float), x0=X[50], xm1=X[50] - d[50]), 60, FS)[0]
    assert rel(y, ref) < 1e-5, rel(y, ref)
    if grad:
        g = (1e3 * rng.normal(size=(1, 90))).astype(np.float32)
        r = OA.reverse(dict(a, Ht=b["Ht"].astype(float)), 90, FS, g[0].astype(float))
        res = sim.grad(90, torch.tensor(g, device="cuda"))
        assert rel(res["row"][0], r["row"]) < 1e-4 and rel(res["x0"][0], r["x0"]) < 1e-4
