"""Timed workloads of the PFC library, from the smallest calls to the largest.

Each case is one thing a program does with the public Python API (the entry points of
``paper_2603_26818_amd``): advance a plain plan by some steps, transform a field, set a state up and
measure it, differentiate a rollout, advance a hydrodynamic, an amplitude or a batched run.  The
values are those of the runs the library is made for: a density of mean r with fluctuations of 0.1
(r between -0.35 and -0.15, dx = pi / 4), normal noise for bare transforms, amplitudes around 0.1.

``exact`` evaluates the documented formulas (include/pfc.h) with torch in 64 bits.
"""
import math

import torch

import paper_2603_26818_amd as pfc

DX = math.pi / 4
TWO_PI = 2.0 * math.pi
# grid lengths with a compiled schedule besides the powers of two: y and the last axis, and x
MIXED = (6, 10, 12, 14, 20, 30, 60, 150, 700, 750, 1400)
MIXED_X = (12, 20, 24, 28, 30, 40, 60, 120, 300, 750, 1400, 1500)

_S3, _R2 = math.sqrt(3.0) / 2.0, 1.0 / math.sqrt(2.0)
LATTICES = {
    "triangular": [(-0.5, -_S3), (1.0, 0.0), (-0.5, _S3)],
    "square": [(1.0, 0.0), (0.0, 1.0)],
    "bcc": [(0.0, _R2, _R2), (0.0, _R2, -_R2), (_R2, 0.0, _R2), (_R2, 0.0, -_R2), (_R2, _R2, 0.0), (_R2, -_R2, 0.0)],
}


def listed():
    return [
        # one step of the 2D 128^2 FP64 run: an interactive loop that looks at the field after every
        # step; the smallest call
        {"name": "step_128x128_f64", "kind": "step", "n": "128x128", "dtype": "f64", "steps": 1, "r": -0.25, "two_mode": False},
        # a 2D film: many steps per call on a grid that fits the caches
        {"name": "step_512x512_f32", "kind": "step", "n": "512x512", "dtype": "f32", "steps": 50, "r": -0.25, "two_mode": False},
        # a slab with the lattice's own periods: every axis another mixed-radix length, two-mode operator
        {"name": "step_150x60x300_f32", "kind": "step", "n": "150x60x300", "dtype": "f32", "steps": 10, "r": -0.2, "two_mode": True},
        # the 256^3 FP64 run
        {"name": "step_256x256x256_f64", "kind": "step", "n": "256x256x256", "dtype": "f64", "steps": 10, "r": -0.3, "two_mode": False},
        # the 512^3 FP32 run (the benchmark's workload)
        {"name": "step_512x512x512_f32", "kind": "step", "n": "512x512x512", "dtype": "f32", "steps": 4, "r": -0.3, "two_mode": False},
        # the paper's own 750^3 grid
        {"name": "step_750x750x750_f32", "kind": "step", "n": "750x750x750", "dtype": "f32", "steps": 2, "r": -0.3, "two_mode": False},
        # bare transforms, there and back: a user's own spectral post-processing
        {"name": "fft_512x512x512_f32", "kind": "fft", "n": "512x512x512", "dtype": "f32"},
        # start of a run and its first measurement: state, energy and mean, structure factor
        {"name": "observe_256x256x256_f32", "kind": "observe", "n": "256x256x256", "dtype": "f32", "r": -0.3, "two_mode": False},
        # density and velocity together, the multiphysics run
        {"name": "hydro_512x512x512_f32", "kind": "hydro", "n": "512x512x512", "dtype": "f32", "steps": 2, "r": -0.3},
        # six coupled bcc amplitudes
        {"name": "apfc_256x256x256_bcc_f32", "kind": "apfc", "n": "256x256x256", "dtype": "f32", "steps": 2, "lattice": "bcc"},
        # a parameter study: 48 independent 2D runs of mixed sizes in one launch
        {"name": "batch_48_f32", "kind": "batch", "sizes": "128,256,512,1024", "each": 12, "dtype": "f32", "steps": 10},
        # a training step: loss on psi(T), gradients of psi0 and r through a checkpointed rollout
        {"name": "rollout_512x512_f32", "kind": "rollout", "n": "512x512", "dtype": "f32", "steps": 50, "r": -0.25, "every": 25},
    ]


def _steps(rng, points, cap):
    """1 .. 50 steps, spread over their logarithm, with points * steps <= cap."""
    hi = max(1, min(50, cap // points))
    return int(round(math.exp(rng.uniform(0.0, math.log(hi))))) if hi > 1 else 1


def _grid(rng, ndim, lo, hi, cap, odd):
    """A grid of ndim axes of lengths lo .. hi with at most cap points; odd: mixed-radix lengths too."""
    while True:
        n = []
        for a in range(ndim):
            pool = [2 ** k for k in range(2, 12) if lo <= 2 ** k <= hi]
            if odd:
                pool += [m for m in (MIXED_X if a == ndim - 1 else MIXED) if lo <= m <= hi]
            pool.sort()
            n.append(pool[int(rng.random() * len(pool))])
        if math.prod(n) <= cap:
            return n


def draw(rng):
    kind = rng.choice(["step", "step", "step3", "step3", "step3", "fft", "observe", "hydro", "apfc", "batch", "rollout"])
    dtype = rng.choice(["f32", "f32", "f64"])
    half = 2 if dtype == "f64" else 1
    r = round(rng.uniform(-0.35, -0.15), 4)
    if kind == "step":
        n = _grid(rng, 2, 32, 2048, 2 ** 22, rng.random() < 0.4)
        return {"kind": "step", "n": "x".join(map(str, n)), "dtype": dtype, "steps": _steps(rng, math.prod(n), 2 ** 27), "r": r,
                "two_mode": rng.random() < 0.3}
    if kind == "step3":
        n = _grid(rng, 3, 12, 1024, 2 ** 28 // half, rng.random() < 0.4)
        return {"kind": "step", "n": "x".join(map(str, n)), "dtype": dtype, "steps": _steps(rng, math.prod(n), 2 ** 29 // half), "r": r,
                "two_mode": rng.random() < 0.3}
    if kind == "fft":
        n = _grid(rng, rng.choice([2, 3]), 12, 1024, 2 ** 28 // half, rng.random() < 0.3)
        return {"kind": "fft", "n": "x".join(map(str, n)), "dtype": dtype}
    if kind == "observe":
        n = _grid(rng, rng.choice([2, 3]), 12, 512, 2 ** 27 // half, rng.random() < 0.3)
        return {"kind": "observe", "n": "x".join(map(str, n)), "dtype": dtype, "r": r, "two_mode": rng.random() < 0.3}
    if kind == "hydro":
        n = _grid(rng, rng.choice([2, 3, 3]), 16, 512, 2 ** 26 // half, rng.random() < 0.3)
        return {"kind": "hydro", "n": "x".join(map(str, n)), "dtype": dtype, "steps": _steps(rng, math.prod(n), 2 ** 27 // half), "r": r}
    if kind == "apfc":
        lattice = rng.choice(["triangular", "square", "bcc"])
        n = _grid(rng, 3 if lattice == "bcc" else 2, 32, 256 if lattice == "bcc" else 1024, 2 ** 24 // half, False)
        return {"kind": "apfc", "n": "x".join(map(str, n)), "dtype": dtype, "steps": _steps(rng, math.prod(n), 2 ** 25 // half),
                "lattice": lattice}
    if kind == "batch":
        sizes = sorted(rng.sample([32, 64, 128, 256, 512, 1024], rng.randint(1, 4)))
        return {"kind": "batch", "sizes": ",".join(map(str, sizes)), "each": rng.randint(1, 12), "dtype": dtype, "steps": rng.randint(1, 10)}
    n = _grid(rng, 2, 32, 512, 2 ** 18, rng.random() < 0.3)
    return {"kind": "rollout", "n": "x".join(map(str, n)), "dtype": dtype, "steps": rng.randint(5, 50), "r": r, "every": rng.choice([10, 25, 50])}


# ---------------------------------------------------------------------------------------- inputs

def _shape(case):
    return tuple(int(v) for v in case["n"].split("x"))


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _device():
    return torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")


def _uniform(g, shape, lo, hi, dtype):
    return torch.empty(shape, dtype=dtype, device=g.device).uniform_(lo, hi, generator=g)


def _params(case):
    """Model parameters of a case (two-mode: the operator with Q1^2 = 2, R1 = 0.05)."""
    two = bool(case.get("two_mode", False))
    return dict(r=float(case.get("r", -0.25)), dt=0.25 if two else 0.5, model=1 if two else 0, q1sq=2.0 if two else 4.0 / 3.0,
                R1=0.05 if two else 0.0)


def _batch_instances(case):
    """each runs per size: one-mode and two-mode in turn, r spread over -0.35 .. -0.15."""
    out = []
    for n in (int(v) for v in case["sizes"].split(",")):
        for j in range(case["each"]):
            two = j % 2 == 1
            out.append(dict(shape=(n, n), dtype=case["dtype"], model=1 if two else 0, r=-0.35 + 0.2 * (j + 0.5) / case["each"], dt=0.25,
                            q1sq=2.0 if two else 4.0 / 3.0, R1=0.05 if two else 0.0))
    return out


def _inputs(case, seed):
    """The input tensors of a case, from the seed alone."""
    kind, dtype = case["kind"], _dtype(case)
    g = torch.Generator(device=_device()).manual_seed(int(seed))
    if kind == "batch":
        return [_uniform(g, i["shape"], i["r"] - 0.1, i["r"] + 0.1, dtype) for i in _batch_instances(case)]
    shape = _shape(case)
    if kind == "fft":
        return torch.empty(shape, dtype=dtype, device=g.device).normal_(generator=g)
    if kind == "apfc":
        n = (len(LATTICES[case["lattice"]]),) + shape
        return torch.complex(_uniform(g, n, 0.05, 0.15, dtype), _uniform(g, n, -0.05, 0.05, dtype))
    r = float(case["r"])
    psi = _uniform(g, shape, r - 0.1, r + 0.1, dtype)
    if kind == "hydro":
        return psi, _uniform(g, (len(shape),) + shape, -0.05, 0.05, dtype)
    if kind == "rollout":
        return psi, _uniform(g, shape, r - 0.1, r + 0.1, dtype)
    return psi


HYDRO = dict(rho0=1.0, gamma=1.0, a0=2.0)
APFC = dict(dB=-0.15, Bx=1.0, t=0.3, v=1.0, dt=0.5, dx=math.pi / 2)


def prepare(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    s = {"kind": kind, "case": case}
    if kind == "batch":
        inst = _batch_instances(case)
        # every run's field is a piece of one array, as its state is
        sizes = [p.numel() for p in x]
        psi = torch.cat([p.reshape(-1) for p in x])
        state = torch.zeros(psi.numel() // 2, dtype=torch.complex128 if case["dtype"] == "f64" else torch.complex64, device=psi.device)
        off = [sum(sizes[:i]) for i in range(len(sizes) + 1)]
        psis = [psi[off[i]:off[i + 1]].view(inst[i]["shape"]) for i in range(len(inst))]
        states = [state[off[i] // 2:off[i + 1] // 2].view(inst[i]["shape"][0], inst[i]["shape"][1] // 2) for i in range(len(inst))]
        s["batch"] = pfc.Batch(inst)
        s["batch"].bind(psis, states)
        s["batch"].state_init()
        s["psi"], s["state"] = psi, state
        return s
    if kind == "apfc":
        s["model"] = pfc.Apfc(_shape(case), LATTICES[case["lattice"]], dtype=case["dtype"], **APFC)
        s["eta"] = x
        s["eta_hat"] = s["model"].state_init(x)
        return s
    plan = s["plan"] = pfc.Plan(_shape(case), dtype=case["dtype"], dx=DX, **_params(case))
    if kind == "fft":
        s["x"] = x
    elif kind == "observe":
        s["psi"] = x
        s["state"] = plan.empty_state().zero_()
    elif kind == "step":
        s["psi"] = x
        s["state"] = plan.state_init(x, plan.empty_state().zero_())
    elif kind == "rollout":
        s["psi"], s["target"] = x
    elif kind == "hydro":
        s["psi"], s["v"] = x
        d = len(plan.shape)
        s["psi_state"] = plan.empty_state().zero_()
        s["v_state"] = torch.zeros((d,) + tuple(plan.state_shape), dtype=plan.complex_dtype, device=plan.device)
        plan.hydro_state_init(s["psi"], s["v"], s["psi_state"], s["v_state"])
        s["work"] = torch.empty(int(pfc.load_library().pfc_hydro_work_bytes(plan._h)), dtype=torch.uint8, device=plan.device)
    return s


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "step":
        return s["plan"].step(s["psi"], s["state"], case["steps"])
    if kind == "fft":
        half = s["plan"].fft_r2c(s["x"])
        return half, s["plan"].fft_c2r(half)
    if kind == "observe":
        state = s["plan"].state_init(s["psi"], s["state"])
        energy = s["plan"].energy(s["psi"], state)
        return energy, s["plan"].state_export(state)
    if kind == "hydro":
        return s["plan"].hydro_step(s["psi"], s["psi_state"], s["v"], s["v_state"], nsteps=case["steps"], work=s["work"], **HYDRO)
    if kind == "apfc":
        return s["model"].step(s["eta"], s["eta_hat"], case["steps"])
    if kind == "batch":
        s["batch"].step(case["steps"])
        return s["psi"], s["state"]
    return pfc.loss_and_grad(s["plan"], s["psi"], float(case["r"]), s["target"], case["steps"], case["every"])


# ---------------------------------------------------------------------------------------- work

def _fft_flops(points):
    return 2.5 * points * math.log2(points)  # one real transform


def work(case):
    """Inputs read once and outputs written once per step (per call where nothing is stepped)."""
    kind = case["kind"]
    b = 8 if case["dtype"] == "f64" else 4
    if kind == "batch":
        pts = [i["shape"][0] * i["shape"][1] for i in _batch_instances(case)]
        return {"bytes": case["steps"] * 4.0 * b * sum(pts), "flops": case["steps"] * sum(2 * _fft_flops(p) + 15.0 * p for p in pts)}
    shape = _shape(case)
    pts = math.prod(shape)
    d = len(shape)
    half = pts // shape[-1] * (shape[-1] // 2 + 1) * 2 * b
    if kind == "step":
        return {"bytes": case["steps"] * 4.0 * b * pts, "flops": case["steps"] * (2 * _fft_flops(pts) + 15.0 * pts)}
    if kind == "fft":
        return {"bytes": 2.0 * (b * pts + half), "flops": 2 * _fft_flops(pts)}
    if kind == "observe":
        return {"bytes": 2.0 * b * pts + half, "flops": _fft_flops(pts) + 15.0 * pts}
    if kind == "hydro":
        return {"bytes": case["steps"] * 2.0 * (2 + 2 * d) * b * pts, "flops": case["steps"] * ((4 + 4 * d) * _fft_flops(pts) + 40.0 * d * pts)}
    if kind == "apfc":
        n = len(LATTICES[case["lattice"]])
        return {"bytes": case["steps"] * 4.0 * n * 2 * b * pts, "flops": case["steps"] * n * (4 * _fft_flops(pts) + 60.0 * pts)}
    # rollout: forward, the replay of it, and one adjoint step (psi_n, psi_n+1, lambda in and out) each
    return {"bytes": case["steps"] * 12.0 * b * pts, "flops": case["steps"] * (7 * _fft_flops(pts) + 45.0 * pts)}


# ---------------------------------------------------------------------------------------- exact

def _modes(shape, device, dx=DX, half=True):
    """Signed wavenumber of every axis, each shaped to broadcast over the (half) spectrum."""
    out = []
    for a, n in enumerate(shape):
        last = half and a == len(shape) - 1
        m = torch.fft.rfftfreq(n, 1.0 / n, dtype=torch.float64, device=device) if last else torch.fft.fftfreq(
            n, 1.0 / n, dtype=torch.float64, device=device)
        out.append((m * (TWO_PI / (n * dx))).view([-1 if i == a else 1 for i in range(len(shape))]))
    return out


def _lap(shape, device):
    q = 0.0
    for k in _modes(shape, device):
        q = q + k * k
    return q


def _corr(p, q):
    return (1 - q) ** 2 * ((p["q1sq"] - q) ** 2 + p["R1"]) if p["model"] else (1 - q) ** 2


def _steps_exact(p, psi, nsteps):
    """psi and its half spectrum after nsteps steps of the plain model."""
    dims = tuple(range(psi.dim()))
    q = _lap(psi.shape, psi.device)
    den = 1 + p["dt"] * q * (p["r"] + _corr(p, q))
    S = torch.fft.rfftn(psi, dim=dims)
    for _ in range(nsteps):
        N = torch.fft.rfftn(psi * psi * psi, dim=dims)
        S = (S - p["dt"] * q * N) / den
        psi = torch.fft.irfftn(S, s=psi.shape, dim=dims)
    return psi, S


def _folded(S):
    """2D half spectrum -> the state's rows of n_x / 2 values, columns 0 and n_x / 2 in one."""
    out = S[:, :-1].clone()
    out[:, 0] = S[:, 0] + 1j * S[:, -1]
    return out


def _exact_hydro(case, psi, v):
    p, h, dims = _params(case), HYDRO, tuple(range(psi.dim()))
    shape, dev = psi.shape, psi.device
    q = _lap(shape, dev)
    lin = p["r"] + _corr(p, q)
    ks = []
    for a, k in enumerate(_modes(shape, dev)):
        k = k.clone()
        k.view(-1)[shape[a] // 2] = 0.0  # no first derivative at a Nyquist index
        ks.append(k)
    inv = lambda X: torch.fft.irfftn(X, s=shape, dim=dims)  # noqa: E731
    fwd = lambda x: torch.fft.rfftn(x, dim=dims)  # noqa: E731
    S, V = fwd(psi), [fwd(c) for c in v]
    v = list(v)
    c = p["dt"] / h["rho0"]
    for _ in range(case["steps"]):
        adv = sum(v[j] * inv(1j * ks[j] * S) for j in range(len(shape)))
        S = (S + p["dt"] * (-q * fwd(psi ** 3) - fwd(adv))) / (1 + p["dt"] * q * lin)
        psi = inv(S)
        mu = fwd(psi ** 3) + lin * S
        for j in range(len(shape)):
            V[j] = (V[j] - c * torch.exp(-0.5 * h["a0"] ** 2 * q) * fwd(psi * inv(1j * ks[j] * mu))) / (1 + c * h["gamma"] * q)
            v[j] = inv(V[j])
    if len(shape) == 2:
        return psi, _folded(S), torch.stack(v), torch.stack([_folded(x) for x in V])
    return psi, None, torch.stack(v), None


def _exact_apfc(case, eta):
    kv, a = LATTICES[case["lattice"]], APFC
    N, dims, shape = len(kv), tuple(range(1, eta.dim())), eta.shape[1:]
    sig = [s for f in range(1, N + 1) for s in (f, -f)]
    vec = {s: [math.copysign(1.0, s) * c for c in kv[abs(s) - 1]] for s in sig}

    def hits(j, *t):
        return all(abs(sum(vec[s][i] for s in t) - kv[j][i]) < 1e-9 for i in range(len(kv[j])))

    products = []  # per field: sorted index tuple -> number of its resonant orders
    for j in range(N):
        m = {}
        for x in sig:
            for y in sig:
                if hits(j, x, y):
                    m[tuple(sorted((x, y)))] = m.get(tuple(sorted((x, y))), 0) + 1
                for z in sig:
                    if hits(j, x, y, z):
                        m[tuple(sorted((x, y, z)))] = m.get(tuple(sorted((x, y, z))), 0) + 1
        products.append(m)
    ks = _modes(shape, eta.device, a["dx"], half=False)
    hat = torch.fft.fftn(eta, dim=dims)
    for _ in range(case["steps"]):
        out = torch.empty_like(eta)
        for j in range(N):
            acc = torch.zeros_like(eta[j])
            for t, mult in products[j].items():
                z = (-a["t"] if len(t) == 2 else a["v"]) * mult
                for s in t:
                    z = z * (eta[s - 1] if s > 0 else eta[-s - 1].conj())
                acc += z
            kk = sum(c * c for c in kv[j])
            G = 1 - sum((k + c) ** 2 for k, c in zip(ks, kv[j]))
            out[j] = (hat[j] - a["dt"] * kk * torch.fft.fftn(acc)) / (1 + a["dt"] * kk * (a["dB"] + a["Bx"] * G * G))
        hat = out
        eta = torch.fft.ifftn(hat, dim=dims)
    return eta, hat


def _exact_rollout(case, psi, target):
    p = _params(case)
    psi0 = psi.clone().requires_grad_(True)
    r = torch.tensor(float(case["r"]), dtype=torch.float64, device=psi.device, requires_grad=True)
    q = _lap(psi.shape, psi.device)
    A = 1 / (1 + p["dt"] * q * (r + _corr(p, q)))
    inv = lambda X: torch.fft.irfftn(X, s=psi.shape, dim=(0, 1))  # noqa: E731
    x = psi0
    for _ in range(case["steps"]):
        x = inv(A * (torch.fft.rfftn(x, dim=(0, 1)) - p["dt"] * q * torch.fft.rfftn(x ** 3, dim=(0, 1))))
    L = ((x - target) ** 2).sum()
    gx, gr = torch.autograd.grad(L, (psi0, r))
    return float(L.detach()), gx, float(gr)


def exact(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    if kind == "batch":
        done = [_steps_exact(i, psi.double(), case["steps"]) for i, psi in zip(_batch_instances(case), x)]
        return torch.cat([psi.reshape(-1) for psi, _ in done]), torch.cat([_folded(S).reshape(-1) for _, S in done])
    if kind == "apfc":
        return _exact_apfc(case, x.to(torch.complex128))
    if kind == "hydro":
        return _exact_hydro(case, x[0].double(), x[1].double())
    if kind == "rollout":
        return _exact_rollout(case, x[0].double(), x[1].double())
    x = x.double()
    dims = tuple(range(x.dim()))
    if kind == "fft":
        half = torch.fft.rfftn(x, dim=dims)
        return half, x
    p = _params(case)
    if kind == "observe":
        S = torch.fft.rfftn(x, dim=dims)
        q = _lap(x.shape, x.device)
        w = torch.full((x.shape[-1] // 2 + 1,), 2.0, dtype=torch.float64, device=x.device)
        w[0] = w[-1] = 1.0
        quad = (w * (p["r"] + _corr(p, q)) * (S.real ** 2 + S.imag ** 2)).sum() / (2.0 * x.numel())
        F = DX ** x.dim() * (quad + (x ** 4).sum() / 4)
        return torch.stack([F, x.mean()]), S
    psi, S = _steps_exact(p, x, case["steps"])
    return psi, _folded(S) if x.dim() == 2 else None
