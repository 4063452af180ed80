"""The work that users of this framework have it do, as cases that can be timed
and compared: time stepping of strings, single plates, uneven batches of plates
and groups of plates that share a tensor, linear strings in closed form,
gradients of the time loop for physical parameters and for coupling tensors,
training of the proposal network, and transfer-function responses with their
gradients.

``prepare`` makes what a program holds before the call (contexts, weights,
targets), ``run`` is one pass through the public entry points, ``exact`` the
same result in 64 bits by plain torch, and ``work`` what the pass cannot do
without.  Every pass starts from the initial state or the initial weights, so
that a pass can be repeated.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_05940_amd import fit, modal, physics, transfer
from paper_2505_05940_amd.mlp import MLP

FS = 44100.0
NET = [1024, 512, 512, 512, 512, 5]  # the proposal network


def listed():
    return [
        # one block of a single string played in real time: the smallest call,
        # a note started and its first 64 samples
        dict(name="string block", kind="strings", modes=30, batch=1, steps=64, scheme="sv", forced=True),
        # the training set of the string proposal: many short strings at once
        dict(name="string batch", kind="strings", modes=12, batch=4096, steps=2205, scheme="sv", forced=False),
        # the single plate, one second of sound (clamped in-plane family)
        dict(name="plate 40", kind="plate", modes=40, family="clamped", steps=44100, scheme="sv", forced=False),
        # the largest plate of the paper's sweep over mode counts, a quarter
        # of a second
        dict(name="plate 100", kind="plate", modes=100, family="sine", steps=11025, scheme="sv", forced=False),
        # the headline batch (plates of 50 to 400 modes), half of its plates
        dict(name="plate batch", kind="plates", lo=50, hi=400, batch=128, steps=221),
        # the training set of the plate proposal: plates of one tensor up to
        # per-row scales
        dict(name="plate group", kind="group", modes=40, batch=16384, steps=441),
        # linear strings over one second, one in eight driven by a force
        dict(name="linear strings", kind="linear", modes=100, batch=2048, steps=44100, forced=256),
        # one iteration of a fit of 64 plates over a quarter of a second
        dict(name="fit 64 plates", kind="fit", modes=40, batch=64, steps=11025),
        # the gradient of one large plate, a tenth of a second
        dict(name="gradient 200", kind="fit", modes=200, batch=1, steps=4410),
        # one iteration of a coupling-tensor fit from one start, a tenth of
        # the paper's 17640 samples and more
        dict(name="tensor fit", kind="tensor", modes=40, batch=1, steps=4410),
        # an epoch of the proposal network's training, 32 batches of 1024
        dict(name="network epoch", kind="train", rows=1024, steps=32),
        # the response of a string's transfer function and its gradient, as an
        # iteration of a transfer-function fit takes them
        dict(name="transfer function", kind="transfer", modes=40, freqs=512, batch=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["strings", "strings", "plate", "plate", "plates", "group", "linear", "fit", "tensor", "train",
                       "transfer"])
    if kind == "strings":
        batch = _log(rng, 1, 4096)
        return dict(kind=kind, modes=_log(rng, 5, 120) if batch < 256 else _log(rng, 5, 30), batch=batch,
                    steps=min(_log(rng, 64, 22050), 4096 * 2205 // batch), scheme=rng.choice(["sv", "sv", "tf"]),
                    forced=rng.random() < 0.5)
    if kind == "plate":
        family = rng.choice(["sine", "sine", "clamped"])
        modes = _log(rng, 8, 128 if family == "sine" else 56)
        return dict(kind=kind, modes=modes, family=family, steps=_log(rng, 441, 44100 if modes <= 60 else 11025),
                    scheme=rng.choice(["sv", "sv", "tf"]), forced=rng.random() < 0.5)
    if kind == "plates":
        lo = _log(rng, 30, 90)
        return dict(kind=kind, lo=lo, hi=rng.randint(lo + 40, 380), batch=_log(rng, 12, 100), steps=_log(rng, 64, 221))
    if kind == "group":
        return dict(kind=kind, modes=rng.randint(20, 64), batch=_log(rng, 512, 12000), steps=_log(rng, 64, 441))
    if kind == "linear":
        batch = _log(rng, 1, 2048)
        return dict(kind=kind, modes=rng.randint(20, 100), batch=batch, steps=_log(rng, 2205, 44100),
                    forced=rng.randint(0, batch // 8))
    if kind == "fit":
        modes = _log(rng, 16, 180)
        if modes > 64:
            return dict(kind=kind, modes=modes, batch=1, steps=_log(rng, 441, 4410))
        return dict(kind=kind, modes=modes, batch=_log(rng, 1, 48), steps=_log(rng, 441, 8820))
    if kind == "tensor":
        return dict(kind=kind, modes=rng.randint(16, 48), batch=_log(rng, 1, 8), steps=_log(rng, 441, 4410))
    if kind == "train":
        return dict(kind=kind, rows=_log(rng, 128, 1024), steps=rng.randint(4, 32))
    return dict(kind=kind, modes=rng.randint(10, 80), freqs=rng.randint(100, 700), batch=_log(rng, 1, 8))


# ------------------------------------------------------------------ inputs
def _rng(case, seed):
    return np.random.default_rng([seed, sum(map(ord, case["kind"]))])


def _noise(rng, n):
    """A force signal: a short noise burst."""
    return rng.normal(size=n).astype(np.float32)


def _strings(case, seed):
    """Kirchhoff-Carrier strings from the priors of the string fits, as
    instance dicts; high modes decay faster."""
    rng = _rng(case, seed)
    n, out = case["modes"], []
    setup = fit.StringSetup(n_modes=n, proj_cells=1024)
    for b in range(case["batch"]):
        spread = 10.0 ** rng.uniform(-0.5, 0.5, size=4)
        L = float(rng.choice(np.linspace(0.5, 0.8, 64)))
        # T0^ kept low for many modes: the top mode stays below the audio band's end
        top = min(1.0, (15.0 / n) ** 2)
        theta = (1e5 * spread[0] * top, 0.2 * top * top, L, spread[2], 6e-3 * top * spread[3])
        inst = fit.string_instance(setup, theta)
        inst["x0"] = 0.5 * inst["x0"]
        inst["xm1"] = inst["x0"].copy()
        inst["kappa"] = inst["kappa"] * top  # the tension force of the high modes within the scheme's stability
        if case["forced"]:
            k = np.arange(1, n + 1)
            inst["b_ext"] = 20.0 * np.sin(k * np.pi * rng.uniform(0.1, 0.9))
            inst["e_ext"] = _noise(rng, 1000)
        out.append(inst)
    return out


def _plate(case, seed):
    """The single steel plate, struck (and driven, when asked) at random places."""
    rng = _rng(case, seed)
    h, Lx, Ly = 1e-3, 0.4, 0.3
    amp = rng.uniform(0.5, 3.0) * h
    (cx, cy), (ox, oy) = rng.uniform(0.1, 0.9, size=2), rng.uniform(0.1, 0.9, size=2)
    wl = dict(inplane=case["family"], Lx=Lx, Ly=Ly, h=h, T0=0.0, E=2e11, nu=0.3, rho=7860.0, n_t=case["modes"],
              n_in=case["modes"], grid=(200, 150) if case["family"] == "clamped" else None,
              damping=("affine_omega", 1.0, 0.002),
              strike=dict(xc=cx * Lx, yc=cy * Ly, amplitude=amp, radius=0.1 * Ly), out=(ox * Lx, oy * Ly),
              proj_grid=(200, 150))
    inst = physics.plate_instance(wl)
    if case["forced"]:
        inst["b_ext"] = 10.0 * rng.normal(size=case["modes"])
        inst["e_ext"] = _noise(rng, 2000)
    return [inst]


def _plates(case, seed):
    """Uneven plates whose highest mode sits at 5 kHz, sine in-plane family."""
    rng = _rng(case, seed)
    out = []
    for b in range(case["batch"]):
        n = int(rng.integers(case["lo"], case["hi"] + 1))
        h = float(rng.uniform(0.5e-3, 2e-3))
        cx, cy, ox, oy = (float(v) for v in rng.uniform(0.1, 0.9, size=4))
        out.append(physics.plate_instance(dict(
            inplane="sine", grid=None, aspect=float(rng.uniform(0.5, 1.0)), top_mode_hz=5000.0, h=h,
            E=float(2e11 * 10.0 ** rng.uniform(-0.5, 0.5)), nu=0.3, rho=7860.0, T0=float(10.0 ** rng.uniform(1.0, 2.0)),
            n_t=n, n_in=n, damping=("affine_omega", 1.0, 0.002),
            strike_rel=dict(xc=cx, yc=cy, amplitude=float(rng.uniform(0.5, 3.0)) * h, radius_rel=0.1),
            out_rel=(ox, oy), proj_grid=(96, 96))))
    return out


def _base():
    """Centre of the plate priors (T0^, D^, a, d1^, d3^): steel, 1 mm, 50 N/m,
    a 5 kHz mode decaying at about 50 /s."""
    rs = 7860.0 * 1e-3
    T0, D = 50.0 / rs, 2e11 * 1e-9 / (12 * (1 - 0.09)) / rs
    w = 2 * np.pi * 5000.0
    lam = (-T0 + math.sqrt(T0 * T0 + 4 * D * w * w)) / (2 * D)
    return np.array([T0, D, 0.75, 1.0, 49.0 / lam])


def _thetas(case, seed):
    """Plate parameters from the priors: one decade for the positive ones, a
    grid of aspect ratios (a tenth of the spread for a lone large plate)."""
    rng = _rng(case, seed)
    base, B = _base(), case["batch"]
    th = np.tile(base, (B, 1))
    for i in (0, 1, 3, 4):
        th[:, i] *= 10.0 ** rng.uniform(-0.5, 0.5, B)
    th[:, 2] = rng.choice(np.linspace(0.5, 1.0, 64), B)
    if case["modes"] > 64:
        th = base * (th / base) ** 0.1
    return th


_SETUPS = {}


def _setup(modes):
    if modes not in _SETUPS:
        _SETUPS[modes] = fit.PlateSetup(n_t=modes, n_in=modes, proj_grid=(96, 72))
    return _SETUPS[modes]


def _linear(case, seed):
    """Stiff linear strings: fundamental 80 to 800 Hz, modes below 12 kHz, the
    first ones driven by a noise burst of 1000 samples."""
    rng = _rng(case, seed)
    out = []
    for b in range(case["batch"]):
        f0, B = rng.uniform(80, 800), rng.uniform(0, 1e-4)
        k = np.arange(1, case["modes"] + 1)
        f = k * f0 * np.sqrt(1 + B * k * k)
        k, w = k[f < 12000.0], 2 * np.pi * f[f < 12000.0]
        x0 = 1e-3 * np.sin(k * np.pi * rng.uniform(0.1, 0.4)) / k ** 2
        inst = dict(kind="linear", omega=w, gamma=rng.uniform(0.5, 3.0) + rng.uniform(0.5, 5.0) * 1e-8 * w * w,
                    x0=x0, xm1=x0.copy(), c=np.sin(k * np.pi * rng.uniform(0.5, 0.9)))
        if b < case["forced"]:
            inst["b_ext"] = np.sin(k * np.pi * rng.uniform(0.1, 0.9))
            inst["e_ext"] = 1000.0 * _noise(rng, 1000)
        out.append(inst)
    return out


def _target(case, seed):
    """The sounds that a fit is to match, [batch, steps] in 64 bits: the modes
    of plates near the start, decaying freely."""
    rng = np.random.default_rng([seed, 99])
    th = _thetas(case, seed) * np.exp(rng.uniform(-0.1, 0.1, size=(case["batch"], 5)))
    m, q, _, _ = _setup(case["modes"]).modes
    t = torch.arange(case["steps"], device="cuda", dtype=torch.float64) / FS
    out = []
    for T0, D, a, d1, d3 in th:
        lam = _lam(m, q, a)
        x0, c = _strike(case["modes"], a)
        w, g = (torch.tensor(v, device="cuda") for v in (np.sqrt(D * lam * lam + T0 * lam), d1 + d3 * lam))
        A = torch.tensor(x0 * c, device="cuda")
        out.append((A[:, None] * torch.exp(-g[:, None] * t) * torch.cos(w[:, None] * t)).sum(0))
    return torch.stack(out)


def _symmetric_start(case, seed):
    """Random symmetric tensors with the rms entry of the plate's own, a start
    of a coupling-tensor fit."""
    rng = np.random.default_rng([seed, 7])
    inst = _tensor_plate(case, seed)
    n = case["modes"]
    H = rng.normal(size=(case["batch"], n, n, n))
    H = 0.5 * (H + H.transpose(0, 1, 3, 2))
    # kept small: a random tensor has no plate's order in it
    return inst, (0.3 * H * np.sqrt(np.mean(inst["Ht"].astype(np.float64) ** 2))).astype(np.float32)


def _tensor_plate(case, seed):
    return _plate(dict(kind="tensor", modes=case["modes"], family="sine", forced=False), seed)[0]


def _net(case, seed):
    """He-normal weights, standardised features and normalised parameters."""
    rng = _rng(case, seed)
    parts = []
    for i, j in zip(NET[:-1], NET[1:]):
        parts += [rng.normal(size=i * j, scale=math.sqrt(2.0 / i)), rng.uniform(-0.05, 0.05, size=j)]
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    n = case["rows"] * case["steps"]
    X = torch.randn(n, NET[0], device="cuda", generator=g)
    Z = torch.rand(n, NET[-1], device="cuda", generator=g) * 2 - 1
    order = torch.randperm(n, device="cuda", generator=g)
    return np.concatenate(parts).astype(np.float32), X, Z, order


def _transfer(case, seed):
    """Coefficients (a1, a2, b1, b2, w) of strings' modes, the points of a Bark
    grid in radians per sample, and the upstream gradient."""
    rng = _rng(case, seed)
    n, coef = case["modes"], []
    for b in range(case["batch"]):
        lam = (np.arange(1, n + 1) * np.pi) ** 2
        T0, D = rng.uniform(1e4, 2e5), rng.uniform(0.05, 0.5)
        gam = 0.5 * (rng.uniform(1, 4) + rng.uniform(1e-3, 5e-3) * lam)
        wd = np.sqrt(D * lam * lam + T0 * lam - gam * gam)
        dec = np.exp(-gam / FS)
        b1 = dec * np.sin(wd / FS) / (wd * FS)
        coef.append(np.stack([-2 * dec * np.cos(wd / FS), dec * dec, b1, 0.3 * b1 * rng.normal(size=n),
                              rng.uniform(0.5, 1.5, size=n)], axis=1))
    z = np.linspace(26.81 * 60.0 / 2020.0 - 0.53, 26.81 * 15000.0 / 16960.0 - 0.53, case["freqs"])
    omega = 2 * np.pi * 1960.0 * (z + 0.53) / (26.28 - z) / FS
    g = rng.normal(size=(case["batch"], case["freqs"], 2))
    return np.concatenate(coef), omega, g


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("strings", "plate", "plates", "linear"):
        insts = dict(strings=_strings, plate=_plate, plates=_plates, linear=_linear)[kind](case, seed)
        sim = modal.Sim(insts, FS, scheme=case.get("scheme", "sv"))
        return dict(kind=kind, sim=sim, steps=case["steps"])
    if kind == "group":
        setup = _setup(case["modes"])
        sim = modal.Sim([fit.plate_instance_shared(setup, t) for t in _thetas(case, seed)], FS)
        return dict(kind=kind, sim=sim, steps=case["steps"])
    if kind == "fit":
        # a program's parameters are single-precision tensors; so are their gradients
        theta = torch.tensor(_thetas(case, seed), dtype=torch.float32, requires_grad=True)
        fit.base_tensor(_setup(case["modes"]))
        return dict(kind=kind, theta=theta, target=_target(case, seed).float(), setup=_setup(case["modes"]),
                    steps=case["steps"])
    if kind == "tensor":
        inst, H = _symmetric_start(case, seed)
        sim = modal.Sim([dict(inst, Ht=h) for h in H], FS, flags=modal.FLAG_GRAD)
        g = torch.Generator(device="cuda").manual_seed(int(seed) + 2)
        ybar = torch.randn(case["batch"], case["steps"], device="cuda", generator=g)
        return dict(kind=kind, sim=sim, H=torch.tensor(H, device="cuda"), ybar=ybar, steps=case["steps"])
    if kind == "train":
        w, X, Z, order = _net(case, seed)
        net = MLP(NET, max_batch=case["rows"])
        return dict(kind=kind, net=net, w=w, X=X, Z=Z, order=order, rows=case["rows"], loss=torch.zeros((), device="cuda"))
    coef, omega, g = _transfer(case, seed)
    off = torch.arange(case["batch"] + 1, dtype=torch.int32) * case["modes"]
    return dict(kind=kind, coef=torch.tensor(coef, requires_grad=True), omega=torch.tensor(omega), off=off,
                g=torch.tensor(g), modes=case["modes"])


def run(s):
    kind = s["kind"]
    if kind == "fit":
        s["theta"].grad = None
        y = fit.ModalFn.apply(s["theta"], s["setup"], s["steps"])
        loss = ((y - s["target"]) ** 2).sum(1) / (s["target"] ** 2).sum(1)
        loss.sum().backward()
        return dict(y=y.detach(), loss=loss.detach(), grad=s["theta"].grad)
    if kind == "tensor":
        for b in range(s["H"].shape[0]):
            s["sim"].set_tensor(b, s["H"][b])
        s["sim"].reset()
        y = s["sim"].run(s["steps"])
        return dict(y=y, grad=s["sim"].grad(s["steps"], s["ybar"], tensor=True)["H"])
    if kind == "train":
        s["net"].set_params(s["w"])
        s["loss"].zero_()
        # the last epochs of the schedule: a small learning rate
        s["net"].train_epoch(s["X"], s["Z"], s["order"], s["rows"], 1e-6, loss_acc=s["loss"])
        return dict(weights=s["net"].params(), loss=s["loss"].clone())
    if kind == "transfer":
        s["coef"].grad = None
        H = transfer.TfResponse.apply(s["coef"], s["off"], s["omega"], s["modes"])
        H.backward(s["g"])
        return dict(H=H.detach(), grad=s["coef"].grad)
    s["sim"].reset()
    return s["sim"].run(s["steps"])


# ------------------------------------------------------------------- exact
def _recursion(omega, gamma, scheme):
    """(m, p, r) of d+ = m q + p d + r f, q+ = q + d+ (Sec. 3.2)."""
    T = 1.0 / FS
    if scheme == "tf":
        w = torch.sqrt(omega ** 2 - gamma ** 2)
        e = torch.exp(-gamma * T)
        return -(1 - e) ** 2 - 4 * e * torch.sin(0.5 * w * T) ** 2, e * e, T * e * torch.sin(w * T) / w
    r = T * T / (1 + gamma * T)
    return -r * omega ** 2, (1 - gamma * T) / (1 + gamma * T), r


def _pad(insts, key, n):
    out = np.zeros((len(insts), n))
    for b, i in enumerate(insts):
        v = np.asarray(i[key], dtype=np.float64)
        out[b, :len(v)] = v
    return torch.tensor(out, device="cuda")


def _steps64(insts, steps, scheme, force):
    """The outputs [batch, steps] of the recursion in 64 bits; force(q) is the
    nonlinear modal force."""
    n = max(len(i["omega"]) for i in insts)
    omega = _pad(insts, "omega", n)
    omega = torch.where(omega > 0, omega, torch.full_like(omega, 100.0))
    gamma = _pad(insts, "gamma", n)
    m, p, r = _recursion(omega, torch.where(gamma > 0, gamma, torch.ones_like(gamma)), scheme)
    q, c = _pad(insts, "x0", n), _pad(insts, "c", n)
    d = q - _pad(insts, "xm1", n)
    E = max([len(i["e_ext"]) for i in insts if i.get("e_ext") is not None], default=0)
    b = torch.zeros_like(q)
    e = torch.zeros(len(insts), max(E, 1), dtype=torch.float64, device="cuda")
    for k, i in enumerate(insts):
        if i.get("e_ext") is not None:
            b[k, :len(i["omega"])] = torch.tensor(np.asarray(i["b_ext"]), device="cuda")
            e[k, :len(i["e_ext"])] = torch.tensor(i["e_ext"].astype(np.float64), device="cuda")
    y = torch.empty(steps, len(insts), dtype=torch.float64, device="cuda")
    for s in range(steps):
        torch.sum(c * q, 1, out=y[s])
        f = force(q)
        if s < E:
            f = f - b * e[:, s:s + 1]
        d = m * q + p * d - r * f
        q = q + d
    return y.T.contiguous()


def _plate_force(H):
    """F(q) of tensors H [batch, rows, modes, modes] in 64 bits."""
    B, R, N, _ = H.shape
    H2 = H.reshape(B, R * N, N)

    def force(q):
        V = (H2 @ q[:, :, None]).reshape(B, R, N)
        eta = (V @ q[:, :, None])
        return (eta * V).sum(1)
    return force


def _lam(m, q, a, area=0.12):
    return np.pi ** 2 * (m ** 2 * a / area + q ** 2 / (a * area))


def _strike(modes, a):
    """Strike projection and pickup weights of a fitted plate at aspect a."""
    m, q, _, _ = _setup(modes).modes
    Lx, Ly = math.sqrt(0.12 / a), math.sqrt(0.12 * a)
    nx, ny = 96, 72
    x, y = (np.arange(nx) + 0.5) * (Lx / nx), (np.arange(ny) + 0.5) * (Ly / ny)
    rad, rr = np.hypot(x[:, None] - 0.37 * Lx, y[None, :] - 0.61 * Ly), 0.1 * min(Lx, Ly)
    w = np.where(rad < rr, 0.5e-3 * (1 + np.cos(np.pi * rad / rr)), 0.0)
    S = np.sin(np.outer(m, x) * (np.pi / Lx)) @ w
    x0 = (S * np.sin(np.outer(q, y) * (np.pi / Ly))).sum(1) * 2 / math.sqrt(0.12) * 0.12 / (nx * ny)
    c = 2 / math.sqrt(0.12) * np.sin(m * np.pi * 0.71) * np.sin(q * np.pi * 0.29)
    return x0, c


def _sine_tensor(modes):
    """Unscaled coupling tensor of the sine in-plane family in closed form,
    int Psi_n L(Phi_i, Phi_j) dS on the base plate."""
    m, q, a, b = (torch.tensor(np.asarray(v, dtype=np.float64), device="cuda") for v in _setup(modes).modes)
    Lx, Ly = math.sqrt(0.12 / 0.75), math.sqrt(0.12 * 0.75)

    def s(k, L):  # int_0^L sin(k pi x / L) dx, k whole
        odd = torch.remainder(k, 2) != 0
        return torch.where(odd, 2 * L / (np.pi * torch.where(odd, k, torch.ones_like(k))), torch.zeros_like(k))

    def parts(n, k, L):
        n, i, j = n[:, None, None], k[None, :, None], k[None, None, :]
        minus, plus = s(n + i - j, L) + s(n - i + j, L), s(n + i + j, L) + s(n - i - j, L)
        return (minus - plus) / 4, (minus + plus) / 4

    (sx, cx), (sy, cy) = parts(a, m, Lx), parts(b, q, Ly)
    al, be = m * np.pi / Lx, q * np.pi / Ly
    A = torch.outer(al ** 2, be ** 2) + torch.outer(be ** 2, al ** 2)
    B = 2 * torch.outer(al * be, al * be)
    return (2 / math.sqrt(0.12)) ** 3 * (A * sx * sy - B * cx * cy)


def _exact_fit(case, seed):
    """Outputs, losses and parameter gradients: the state and its derivatives
    by the five parameters stepped together in 64 bits."""
    th = torch.tensor(_thetas(case, seed), dtype=torch.float32).double().numpy()
    n, B, S = case["modes"], case["batch"], case["steps"]
    m, q, ai, bi = _setup(n).modes
    H0 = _sine_tensor(n).reshape(n * n, n)
    dev = dict(device="cuda", dtype=torch.float64)
    om, dom = np.zeros((B, n)), np.zeros((B, n, 5))
    ga, dga = np.zeros((B, n)), np.zeros((B, n, 5))
    sc, dsc = np.zeros((B, n)), np.zeros((B, n, 5))  # squared row scales
    x0, dx0, cc, dcc = np.zeros((B, n)), np.zeros((B, n, 5)), np.zeros((B, n)), np.zeros((B, n, 5))
    for b, (T0, D, a, d1, d3) in enumerate(th):
        lam, zeta = _lam(m, q, a), _lam(ai, bi, a)
        dl = np.pi ** 2 * (m ** 2 / 0.12 - q ** 2 / (a * a * 0.12))
        dz = np.pi ** 2 * (ai ** 2 / 0.12 - bi ** 2 / (a * a * 0.12))
        om[b] = np.sqrt(D * lam * lam + T0 * lam)
        dom[b] = np.stack([lam, lam * lam, (2 * D * lam + T0) * dl, 0 * lam, 0 * lam], 1) / (2 * om[b])[:, None]
        ga[b] = d1 + d3 * lam
        dga[b] = np.stack([0 * lam, 0 * lam, d3 * dl, 1 + 0 * lam, lam], 1)
        sc[b] = 6 * (1 - 0.09) * D / 1e-6 / zeta ** 2
        dsc[b] = np.stack([0 * zeta, sc[b] / D, -2 * sc[b] * dz / zeta, 0 * zeta, 0 * zeta], 1)
        h = 1e-6 * a
        (x0[b], cc[b]), (xp, cp), (xm, cm) = _strike(n, a), _strike(n, a + h), _strike(n, a - h)
        dx0[b, :, 2], dcc[b, :, 2] = (xp - xm) / (2 * h), (cp - cm) / (2 * h)
    om, dom, ga, dga, sc, dsc, x0, dx0, cc, dcc = (torch.tensor(v, **dev) for v in
                                                   (om, dom, ga, dga, sc, dsc, x0, dx0, cc, dcc))
    T = 1 / FS
    k = 1 + ga * T
    r, p = T * T / k, (1 - ga * T) / k
    mm = -r * om ** 2
    dr = -(T * T * T / k ** 2)[..., None] * dga
    dp = -(2 * T / k ** 2)[..., None] * dga
    dm = -dr * (om ** 2)[..., None] - (2 * r * om)[..., None] * dom
    # Q[..., 0] is the state, Q[..., 1:] its derivatives by the parameters
    Q, D = torch.cat([x0[..., None], dx0], 2), torch.zeros(B, n, 6, **dev)
    C = torch.cat([cc[..., None], dcc], 2)
    zero = torch.zeros(B, n, 1, **dev)
    dM, dP, dR, dS = (torch.cat([zero, v], 2) for v in (dm, dp, dr, dsc))
    y = torch.empty(S, B, 6, **dev)
    mm, p, r, sc = mm[..., None], p[..., None], r[..., None], sc[..., None]
    for t in range(S):
        q0 = Q[..., :1]
        Y = cc[..., None] * Q + C * q0
        Y[..., 0] -= (C * q0)[..., 0]
        y[t] = Y.sum(1)
        V = (H0 @ Q.permute(1, 0, 2).reshape(n, B * 6)).reshape(n, n, B, 6).permute(2, 0, 1, 3)  # [B, row, mode, 6]
        V0 = V[..., 0]
        eta = torch.stack([(V0 * q0[:, None, :, 0]).sum(2)], 2)  # [B, row, 1]
        deta = 2 * (V0.transpose(1, 2).contiguous()[..., None] * Q[:, :, None, :]).sum(1)  # [B, row, 6]
        deta[..., 0] = 0
        w = deta * sc + eta * dS
        F = torch.bmm(V0.transpose(1, 2).contiguous(), w) + (V * (eta * sc)[..., None]).sum(1)
        D2 = mm * Q + p * D - r * F + dM * q0 + dP * D[..., :1] - dR * F[..., :1]
        D = D2
        Q = Q + D
    y = y.permute(1, 2, 0)
    tgt = _target(case, seed).float().double()
    norm = (tgt ** 2).sum(1)
    diff = y[:, 0] - tgt
    return dict(y=y[:, 0].contiguous(), loss=(diff ** 2).sum(1) / norm,
                grad=(2 * diff[:, None] * y[:, 1:]).sum(2) / norm[:, None])


def _exact_tensor(case, seed):
    """Outputs and tensor gradients: the recursion and its reverse in 64 bits."""
    inst, H = _symmetric_start(case, seed)
    B, n, S = case["batch"], case["modes"], case["steps"]
    dev = dict(device="cuda", dtype=torch.float64)
    H = torch.tensor(H, **dev)
    H2 = H.reshape(B, n * n, n)
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 2)
    ybar = torch.randn(B, S, device="cuda", generator=g).double()
    omega, gamma, x0, c = (torch.tensor(np.asarray(inst[k]), **dev) for k in ("omega", "gamma", "x0", "c"))
    m, p, r = _recursion(omega, gamma, "sv")
    q, d = x0.repeat(B, 1), torch.zeros(B, n, **dev)
    qs = torch.empty(S, B, n, **dev)
    for t in range(S):
        qs[t] = q
        V = (H2 @ q[:, :, None]).reshape(B, n, n)
        F = ((V @ q[:, :, None]) * V).sum(1)
        d = m * q + p * d - r * F
        q = q + d
    y = (qs * c).sum(2).T.contiguous()
    qb, db = torch.zeros(B, n, **dev), torch.zeros(B, n, **dev)
    us, etas, ws = torch.empty(S, B, n, **dev), torch.empty(S, B, n, **dev), torch.empty(S, B, n, **dev)
    for t in range(S - 1, -1, -1):
        q = qs[t]
        db = qb + p * db
        u = r * db
        VW = (H2 @ torch.stack([q, u], 2)).reshape(B, n, n, 2)
        V, W = VW[..., 0], VW[..., 1]
        eta, w = (V @ q[:, :, None])[..., 0], (V @ u[:, :, None])[..., 0]
        us[t], etas[t], ws[t] = u, eta, w
        qb = ybar[:, t:t + 1] * c + qb + m * db - (2 * w[..., None] * V + eta[..., None] * W).sum(1)
    grad = []
    for b in range(B):
        rows = [-((ws[:, b, i:i + 1] * qs[:, b] + etas[:, b, i:i + 1] * us[:, b]).T @ qs[:, b]) for i in range(n)]
        grad.append(torch.stack(rows))
    return dict(y=y, grad=grad)


def _exact_transfer(case, seed):
    coef, omega, g = _transfer(case, seed)
    n, z = case["modes"], np.exp(1j * omega)[None, :]
    H, grad = [], []
    for b in range(case["batch"]):
        a1, a2, b1, b2, w = (v[:, None] for v in coef[b * n:(b + 1) * n].T)
        den, num = z * z + a1 * z + a2, b1 * z + b2
        h = (w * num / den).sum(0)
        H.append(np.stack([h.real, h.imag], 1))
        gc = (g[b, :, 0] - 1j * g[b, :, 1])[None, :]  # Re(conj(G) dH)
        d = [-w * num * z / den ** 2, -w * num / den ** 2, w * z / den, w / den, num / den]
        grad.append(np.stack([(gc * v).real.sum(1) for v in d], 1))
    return dict(H=np.stack(H), grad=np.concatenate(grad))


def exact(case, seed):
    kind = case["kind"]
    if kind == "strings":
        insts = _strings(case, seed)
        n = case["modes"]
        lam, kappa = _pad(insts, "lam", n), torch.tensor([i["kappa"] for i in insts], device="cuda")[:, None]
        return _steps64(insts, case["steps"], case["scheme"],
                        lambda q: kappa * lam * q * (lam * q * q).sum(1, keepdim=True))
    if kind == "plate":
        insts = _plate(case, seed)
        H = torch.tensor(insts[0]["Ht"], device="cuda").double()[None]
        return _steps64(insts, case["steps"], case["scheme"], _plate_force(H))
    if kind == "plates":
        rows = []
        for inst in _plates(case, seed):
            H = torch.tensor(inst.pop("Ht"), device="cuda").double()[None]
            rows.append(_steps64([inst], case["steps"], "sv", _plate_force(H)))
        return torch.cat(rows)
    if kind == "group":
        th, n = _thetas(case, seed), case["modes"]
        m, q, ai, bi = _setup(n).modes
        H0 = _sine_tensor(n).reshape(n * n, n)
        insts, s2 = [], []
        strikes = {a: _strike(n, a) for a in set(th[:, 2])}
        for T0, D, a, d1, d3 in th:
            lam = _lam(m, q, a)
            x0, c = strikes[a]
            insts.append(dict(omega=np.sqrt(D * lam * lam + T0 * lam), gamma=d1 + d3 * lam, x0=x0, xm1=x0, c=c))
            s2.append(6 * (1 - 0.09) * D / 1e-6 / _lam(ai, bi, a) ** 2)
        s2 = torch.tensor(np.stack(s2), device="cuda")

        def force(x):
            V = (H0 @ x.T).reshape(n, n, -1)  # [row, mode, plate]
            eta = (V * x.T).sum(1) * s2.T
            return (V * eta[:, None]).sum(0).T
        return _steps64(insts, case["steps"], "sv", force)
    if kind == "linear":
        return _steps64(_linear(case, seed), case["steps"], "sv", lambda q: 0.0 * q)
    if kind == "fit":
        return _exact_fit(case, seed)
    if kind == "tensor":
        return _exact_tensor(case, seed)
    if kind == "train":
        return None  # sixteen-bit products: no 64-bit value of the whole training
    return _exact_transfer(case, seed)


# -------------------------------------------------------------------- work
def work(case):
    """Bytes: inputs once, outputs once; a tensor that no chip holds (more than
    256 MB stored by parity blocks, one of each transposed pair) once a
    sample.  Operations: a product and a sum per stored tensor entry and use,
    the forces and updates of the modes."""
    kind, S = case["kind"], case.get("steps", 1)
    if kind in ("strings", "linear"):
        n = case["modes"] * case["batch"]
        return dict(bytes=4.0 * case["batch"] * S + 64.0 * n, flops=20.0 * n * S)
    if kind in ("plate", "plates", "group", "fit", "tensor"):
        if kind == "plates":
            # mean of N^3 over the range
            lo, hi = case["lo"], case["hi"]
            n3, n1 = (hi ** 4 - lo ** 4) / 4.0 / (hi - lo), 0.5 * (lo + hi)
        else:
            n3, n1 = float(case["modes"]) ** 3, float(case["modes"])
        B = case.get("batch", 1)
        held = n3 / 4.0 if kind != "tensor" else n3  # entries that parity leaves
        flops = B * S * (2.0 * held + 4.0 * n1 * n1 + 20.0 * n1)
        if kind == "group":
            return dict(bytes=4.0 * held + B * (4.0 * S + 64.0 * n1 + 4.0 * n1), flops=flops)
        stored = 4.0 * B * held * (0.625 if kind != "tensor" else 0.5)
        bytes_ = stored * (S if stored > 256e6 else 1) + B * (4.0 * S + 64.0 * n1)
        if kind in ("fit", "tensor"):
            flops *= 3.0
            if kind == "tensor":
                flops += 2.0 * B * S * n3
                bytes_ += 4.0 * B * n3
        return dict(bytes=bytes_, flops=flops)
    if kind == "train":
        w = sum(i * j for i, j in zip(NET[:-1], NET[1:]))
        rows = case["rows"] * S
        return dict(bytes=4.0 * rows * (NET[0] + NET[-1]) + 8.0 * w, flops=6.0 * w * rows)
    n = case["modes"] * case["batch"]
    return dict(bytes=80.0 * n + 40.0 * case["batch"] * case["freqs"], flops=100.0 * n * case["freqs"])
