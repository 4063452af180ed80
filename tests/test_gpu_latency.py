"""The latency kernel (von Karman plates of more than 64 modes, few at a time)
against the recursion in numpy FP64: units whole and in slabs, their rows
streamed and in registers (four and eight blocks a wave), forces exchanged
directly and through the slabs that own modes, modes and rows beside the tile
and slab sizes, a batch of different plates, runs in parts and after a reset.

The forces are FP32: sums of at most 260^2 products in random order, relative
error about 1e-6 of a force that moves the state by less than itself over these
runs, so 1e-5; a lost row, slab or mode is of order 1e-2 and more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS, STEPS = 44100.0, 120


def _plate(rng, nt, nin, forced):
    H = rng.normal(size=(nin, nt, nt))
    H = (H + H.transpose(0, 2, 1)) * (4e3 / np.sqrt(nt * nin))
    w = 2 * np.pi * np.sort(rng.uniform(50, 6000, nt))
    p = dict(kind="vk", omega=w, gamma=rng.uniform(0.5, 20, nt), x0=rng.normal(size=nt) / np.sqrt(nt), c=rng.normal(size=nt),
             Ht=H.astype(np.float32))
    p["xm1"] = p["x0"] * 0.98
    if forced:
        p["b_ext"], p["e_ext"] = rng.normal(size=nt), (1e6 * rng.normal(size=STEPS // 2)).astype(np.float32)
    return p


def _ref(p):
    T = 1 / FS
    g, w, H = p["gamma"], p["omega"], p["Ht"].astype(float)
    r = T * T / (1 + g * T)
    x, d, y = p["x0"].copy(), p["x0"] - p["xm1"], []
    moved = 0.
    for n in range(STEPS):
        y.append(p["c"] @ x)
        V = H @ x
        F = (V @ x) @ V
        moved = max(moved, np.abs(r * F).max() / np.abs(x).max())
        e = p["e_ext"][n] if "e_ext" in p and n < len(p["e_ext"]) else 0.
        d = -r * w * w * x + (1 - g * T) / (1 + g * T) * d + r * (p.get("b_ext", 0.) * e - F)
        x = x + d
    return np.array(y), moved


@pytest.mark.parametrize("shapes", [[(65, 3)], [(65, 66)], [(72, 9), (68, 33), (97, 64)], [(100, 101)], [(131, 129)],
                                    [(196, 130)], [(256, 65)], [(257, 40)], [(66, 5)] * 18])
def test_latency_plates(shapes):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(sum(a * b for a, b in shapes))
    plates = [_plate(rng, nt, nin, i % 2 == 0) for i, (nt, nin) in enumerate(shapes)]
    refs = [_ref(p) for p in plates]
    assert all(m > 1e-6 for _, m in refs)
    sim = modal.Sim(plates, FS)
    whole = sim.run(STEPS).cpu().numpy()
    for b, (y, _) in enumerate(refs):
        assert np.linalg.norm(whole[b] - y) < 1e-5 * np.linalg.norm(y), b
    sim.reset()
    parts = [sim.run(k).cpu().numpy() for k in (1, 2, 50, STEPS - 53)]
    assert np.array_equal(np.concatenate(parts, 1), whole)
    sim.close()


@pytest.mark.parametrize("shapes", [[(65, 3)], [(72, 9), (68, 33), (97, 64)], [(131, 129)], [(196, 130)], [(250, 66)],
                                    [(66, 5)] * 18])
def test_latency_gradients(shapes):
    """The reverse step with rows in registers against the streaming reverse
    kernel on an explicit launch shape, every gradient; the same reasoning."""
    import torch
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(sum(a * b for a, b in shapes))
    plates = [_plate(rng, nt, nin, i % 2 == 0) for i, (nt, nin) in enumerate(shapes)]
    ybar = torch.tensor(rng.normal(size=(len(plates), STEPS)), dtype=torch.float32, device="cuda")
    got = []
    for kw in ({}, dict(waves=4, max_workgroups=32)):
        sim = modal.Sim(plates, FS, flags=modal.FLAG_GRAD, **kw)
        got.append([sim.grad(STEPS, ybar, tensor=t) for t in (False, True)])
        sim.close()

    def flat(v):
        v = v if isinstance(v, (list, tuple)) else [v]
        return np.concatenate([np.asarray(a.cpu() if torch.is_tensor(a) else a, dtype=float).ravel() for a in v])

    for a, b in zip(*got):
        assert a.keys() == b.keys()
        for key in a:
            if a[key] is None:
                continue
            x, y = flat(a[key]), flat(b[key])
            assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(y), key
