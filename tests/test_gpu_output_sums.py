"""The output sample is an FP32 sum over the modes, and its error that of the
order of the additions: every kernel adds as a tree.  The first sample of a run
is a sum over the initial state, so it can be compared bit for bit with the
same tree in numpy: the on-chip kernel, the kernel of shared tensors by mode
class, and the latency kernel, at mode counts on and off the sizes of lanes,
quads and waves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FS = 44100.0
F = np.float32


def _fma(a, b, c):
    """FP32 fma: the product is exact in FP64, and rounding the sum twice matters
    once in 2^29 values."""
    return F(np.float64(a) * np.float64(b) + np.float64(c))


def _tree(v, halves=False):
    """Neighbours added pairwise, or (halves) element i to element i + n/2."""
    v = list(v)
    while len(v) > 1:
        n = len(v) // 2
        v = [F(v[i] + v[i + n]) for i in range(n)] if halves else [F(v[2 * i] + v[2 * i + 1]) for i in range(n)]
    return v[0]


def _pad(v, n):
    return np.concatenate([np.asarray(v, F), np.zeros(n - len(v), F)])


def _plate(rng, n, n_in, **kw):
    x0 = rng.normal(size=n)
    return dict(kind="vk", omega=2 * np.pi * np.linspace(60, 9000, n), gamma=np.full(n, 3.0), x0=x0, xm1=x0.copy(),
                c=rng.normal(size=n), Ht=np.zeros((n_in, n, n), F), **kw)


def _first(sim):
    return sim.run(3).cpu().numpy()[:, 0]


def test_on_chip():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(1)
    insts = [_plate(rng, n, 4) for n in [1, 3, 4, 5, 15, 16, 17, 40, 63, 64] * 30]
    y = _first(modal.Sim(insts, FS))
    for b, p in enumerate(insts):
        v = _pad(F(p["c"]) * F(p["x0"]), 64).reshape(16, 4)  # four modes a read
        a = [_tree(v[:, j]) for j in range(4)]
        assert y[b] == F(F(a[0] + a[1]) + F(a[2] + a[3])), (b, len(p["c"]))


def test_shared_by_class():
    import torch
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(2)
    for n in (7, 20, 40, 64):
        cls = (np.arange(n) % 4).astype(np.uint8)
        H = np.zeros((5, n, n), F)
        insts = [dict(_plate(rng, n, 5), Ht=H, mode_class=cls) for _ in range(50)]
        sim = modal.Sim(insts, FS)
        assert sim.info()["path"] == 1
        y = _first(sim)
        for b, p in enumerate(insts):
            c, x = np.zeros(64, F), np.zeros(64, F)
            for q in range(4):  # sixteen slots a class
                c[16 * q:16 * q + np.sum(cls == q)] = p["c"][cls == q]
                x[16 * q:16 * q + np.sum(cls == q)] = p["x0"][cls == q]
            t = [_fma(c[i + 32], x[i + 32], F(c[i] * x[i])) for i in range(32)]  # two slots a thread
            w = [_tree([t[4 * i], t[4 * i + 1], t[4 * i + 2], t[4 * i + 3]], halves=True) for i in range(8)]
            assert y[b] == _tree(w, halves=True), (n, b)


def test_latency():
    import torch
    from paper_2505_05940_amd import modal
    rng = np.random.default_rng(3)
    for n, n_in in [(65, 3), (66, 8), (100, 20), (131, 9), (200, 40), (256, 8), (257, 8), (600, 4)]:
        for _ in range(8):
            p = _plate(rng, n, n_in)
            y = _first(modal.Sim([p], FS))
            c, x = _pad(p["c"], 1024), _pad(p["x0"], 1024)
            quads = []
            for i in range(0, 1024, 4):
                v = F(c[i] * x[i])
                for j in range(1, 4):
                    v = _fma(c[i + j], x[i + j], v)
                quads.append(v)
            nw = 8
            lanes = np.zeros((nw, 16), F)  # sixteen quads a wave, 512 threads' modes after one another
            for k, v in enumerate(quads):
                lanes[k // 16 % nw, k % 16] += v
            assert y[0] == _tree([_tree(w) for w in lanes]), n
