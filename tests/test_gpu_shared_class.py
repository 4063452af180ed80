"""The shared-tensor kernel that holds its tensors in registers by mode class,
at the edges of its tiles: classes of 1, 4, 5 and 16 modes, empty classes,
few and many in-plane rows, rows without entries, part-filled workgroups and
chunks, two groups in one launch, and the shapes on either side of its limit
(17 modes in a class; a row more than the tiles hold), against the FP64 loop.
Bar: 1e-5 relative L2 per output signal, as for the other kernels."""
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


def _group(rng, classes, n_in, batch, forced):
    n = sum(classes)
    cls = rng.permutation(np.repeat(np.arange(4), classes)).astype(np.uint8)
    H = rng.normal(size=(n_in, n, n))
    H = 0.5 * (H + H.transpose(0, 2, 1)) * np.sqrt(4.0 / (n * n_in))
    for i in range(n_in):
        H[i] *= (cls[:, None] ^ cls[None, :]) == rng.integers(4)
    H = (3e6 * H).astype(np.float32)
    om = 2 * np.pi * np.sort(rng.uniform(80, 7000, n))
    out = []
    for b in range(batch):
        x0 = 1e-3 * rng.normal(size=n)
        inst = dict(kind="vk", omega=om * rng.uniform(0.97, 1.03), gamma=rng.uniform(1, 30, n), x0=x0, xm1=x0.copy(),
                    c=rng.normal(size=n), Ht=H, h_row_scale=rng.uniform(0.5, 1.5, n_in), mode_class=cls)
        if b in forced:
            inst.update(b_ext=20 * rng.normal(size=n), e_ext=rng.normal(size=70).astype(np.float32))
        out.append(inst)
    return out


def _check(gpu, insts, picks, steps=100):
    modal, torch = gpu
    sim = modal.Sim(insts, FS)
    assert sim.info()["path"] == 1
    y = torch.cat([sim.run(33), sim.run(steps - 33)], 1).double().cpu().numpy()
    for b in picks:
        i = insts[b]
        ref, X, d, _ = OA.forward(dict(i, Ht=i["Ht"].astype(float) * i["h_row_scale"][:, None, None]), steps + 1, FS)
        assert np.linalg.norm(y[b] - ref[:-1]) <= 1e-5 * np.linalg.norm(ref[:-1]), b
        x, xm = sim.state()
        o = sum(len(k["omega"]) for k in insts[:b])
        assert np.linalg.norm(x[o:o + len(i["omega"])] - X[-1]) <= 1e-5 * np.linalg.norm(X[-1])


@pytest.mark.parametrize("classes,n_in,batch", [((1, 1, 1, 1), 4, 16), ((4, 4, 4, 4), 16, 17), ((5, 3, 2, 1), 50, 40),
                                                ((16, 0, 0, 0), 9, 31), ((9, 10, 10, 11), 40, 33),
                                                ((16, 12, 13, 11), 52, 20), ((8, 0, 8, 3), 64, 16),
                                                ((12, 12, 12, 12), 1, 16), ((17, 12, 11, 10), 30, 16),
                                                ((14, 14, 14, 14), 64, 16)])
def test_class_tiles(gpu, classes, n_in, batch):
    rng = np.random.default_rng(sum(classes) * 100 + n_in)
    _check(gpu, _group(rng, classes, n_in, batch, {0, batch - 1}), sorted({0, 1, 15, batch - 1}))


def test_two_groups(gpu):
    rng = np.random.default_rng(5)
    a, b = _group(rng, (3, 2, 2, 1), 7, 20, {3}), _group(rng, (9, 10, 10, 11), 40, 37, {0})
    _check(gpu, a + b, [0, 3, 19, 20, 36, 56])
