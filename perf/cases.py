"""The work that programs have this library do, as cases that can be timed.

A case names one kind of call (``do``) and its sizes and options:

* ``interp``     values (and the gradient) at scattered positions, one call;
* ``noalloc``    the same through the entry point that allocates nothing;
* ``advance``    the one-shot time stepper on the caller's positions;
* ``resident``   steps of particles kept in the library, then a store of the
                 state in the caller's order (``type``: tracers, ellipsoid axes,
                 inertial particles);
* ``loop``       one step of a solver's loop: the field from its half spectrum,
                 one Heun step with the gradient, a store;
* ``next``       a Heun step between the fields of its two times, a store;
* ``learned``    the learned correction form without its fallback;
* ``batch``      loss and gradient of one training batch of the learned form.

Fields are solenoidal random-phase fields with a k^(-5/3) spectrum up to a
third of the grid's wave numbers, unit rms; particles are uniform in the box,
some of them in periodic images of it (unwrapped trajectories).
"""
import math
from fractions import Fraction

import torch

from paper_2107_01104_amd import ptk

L = 2.0 * math.pi
DEV = "cuda"
STORE = {"f64": ptk.F64, "f32": ptk.F32, "bf16": ptk.BF16, "f16": ptk.F16}
NODE_BYTES = {"f64": 24, "f32": 12, "bf16": 6, "f16": 6}
SCHEMES = {"euler": ptk.EULER, "heun": ptk.HEUN, "ab2": ptk.AB2, "ab3": ptk.AB3, "ab4": ptk.AB4}
ORDER = {"ab2": 2, "ab3": 3, "ab4": 4}
AB = {1: (1.0,), 2: (1.5, -0.5), 3: (23 / 12, -16 / 12, 5 / 12), 4: (55 / 24, -59 / 24, 37 / 24, -9 / 24)}
TAU, SHAPE = 0.1, 0.8  # response time of the inertial particles, shape factor of the ellipsoids
HIDDEN, FEATURES, PITCH = 128, 195, 200


def _case(do, N, np_, family, I, m, storage, **more):
    return dict({"do": do, "N": N, "np": np_, "family": family, "I": I, "m": m, "storage": storage, "grad": False,
                 "scheme": "heun", "nsteps": 1, "dt": 1e-3, "type": "tracers"}, **more)


def listed():
    return [
        # a probe of a small field: latency alone counts
        dict(_case("interp", 32, 1000, "lagrange", 4, 0, "f64"), name="probe_32"),
        # the smallest tracking run: 10^4 tracers on 32^3 in the paper's precision, a step per call
        dict(_case("advance", 32, 10000, "lagrange", 4, 0, "f64"), name="heun_step_32"),
        # a serving loop that may not allocate, on a grid that no tile divides
        dict(_case("noalloc", 100, 20000, "spline", 4, 1, "f32"), name="noalloc_100"),
        # the paper's own density (10^8 particles on 4096^3 are 0.0015 a cell): few tracers on a large grid
        dict(_case("interp", 512, 200003, "spline", 8, 2, "f32", grad=True), name="few_on_512"),
        # 16-bit storage, a prime grid and a ragged count, values and gradients
        dict(_case("interp", 193, 777777, "spline", 6, 2, "bf16", grad=True), name="ragged_193_bf16"),
        # the mid-size run: 256^3, 10^7 particles, C1 I = 6, Adams-Bashforth steps
        dict(_case("resident", 256, 10_000_000, "spline", 6, 1, "f32", scheme="ab2", nsteps=5, dt=2e-3), name="ab2_256"),
        # ellipsoid axes: value and gradient at both Heun stages
        dict(_case("resident", 256, 1_000_000, "spline", 8, 2, "f32", type="axes"), name="axes_256"),
        # the paper's precision throughout, value and gradient
        dict(_case("interp", 512, 12_500_000, "spline", 8, 2, "f64", grad=True), name="f64_grad_512"),
        # the headline run: 1024^3, 10^8 particles, C2 I = 8, a Heun step that returns its gradient
        dict(_case("resident", 1024, 100_000_000, "spline", 8, 2, "f32", grad=True), name="heun_grad_1024"),
        # a solver's loop: the field from the vorticity spectrum every step, then the particles
        dict(_case("loop", 512, 12_500_000, "spline", 8, 2, "f32", grad=True, kind="vorticity", spec="c128"), name="loop_512"),
        # the learned form's inference
        dict(_case("learned", 512, 12_500_000, "spline", 8, 2, "f32"), name="learned_512"),
        # the learned form's training direction: forward and backward of the trainer's largest batch
        dict(_case("batch", 64, 16384, "spline", 8, 2, "f32"), name="batch_16384"),
    ]


KERNELS = [("lagrange", 4, 0), ("spline", 4, 1), ("lagrange", 6, 0), ("spline", 6, 1), ("spline", 6, 2),
           ("lagrange", 8, 0), ("spline", 8, 1), ("spline", 8, 2), ("spline", 8, 2), ("spline", 8, 3)]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    do = rng.choice(["interp", "interp", "interp", "noalloc", "advance", "advance", "resident", "resident", "resident",
                     "loop", "next", "learned", "batch"])
    if do == "batch":
        return _case(do, 64, 64 * int(round(_log(rng, 1, 256))), "spline", 8, 2, "f32")
    N = int(round(_log(rng, 24, 512)))
    family, I, m = rng.choice(KERNELS)
    storage = rng.choice(["f32", "f32", "f32", "f64", "bf16", "f16"])
    # particles per cell: from the paper's 0.0015 to a crowded small grid
    n = int(min(2e7, max(500, N ** 3 * _log(rng, 1e-3, 2.0))))
    c = _case(do, N, n, family, I, m, storage, grad=rng.random() < 0.5)
    if do == "noalloc":
        c.update(np=min(n, 1_000_000), grad=False)
    elif do == "advance" or do == "resident":
        c.update(scheme=rng.choice(["heun", "heun", "euler", "ab2", "ab3", "ab4"]), nsteps=rng.choice([1, 1, 2, 5]))
        if do == "resident":
            c.update(type=rng.choice(["tracers", "tracers", "axes", "inertia"]))
    elif do == "loop":
        if rng.random() < 0.5:  # solvers' grids are mostly powers of two
            c.update(N=rng.choice([64, 128, 256]))
        c.update(N=c["N"] + c["N"] % 2, kind=rng.choice(["vorticity", "vorticity", "velocity"]),
                 spec=rng.choice(["c128", "c128", "c64"]))
        if c["spec"] == "c64":  # a solver in single precision keeps its field in single precision
            c.update(storage="f32")
    elif do == "learned":
        c.update(family="spline", I=8, m=2, storage="f32", grad=False)
    return c


# ---------------------------------------------------------------- inputs

def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 16 + k)
    return g


def _wave_numbers(N, dtype):
    kf = torch.fft.fftfreq(N, d=1.0 / N, device=DEV, dtype=dtype)
    kr = torch.fft.rfftfreq(N, d=1.0 / N, device=DEV, dtype=dtype)
    return kr.view(1, 1, -1), kf.view(1, N, 1), kf.view(N, 1, 1)


def _solenoidal(N, seed, dtype):
    """The three components' half spectra [k3][k2][k1] of a real solenoidal field (from real white noise, so Hermitian)."""
    K = _wave_numbers(N, dtype)
    kk = torch.sqrt(K[0] * K[0] + K[1] * K[1] + K[2] * K[2])
    kc = N / 3.0
    safe = kk.clamp(min=1.0)
    amp = safe ** (-11.0 / 6.0) * torch.exp(-(kk - kc).clamp(min=0.0) / (0.1 * kc))
    amp = torch.where((kk >= 1) & (K[0].abs() < N / 2) & (K[1].abs() < N / 2) & (K[2].abs() < N / 2), amp, torch.zeros_like(amp))
    g = _gen(seed, 0)
    w = []
    for _ in range(3):
        w.append(torch.fft.rfftn(torch.randn((N, N, N), generator=g, device=DEV, dtype=dtype)))
    kdot = (K[0] * w[0] + K[1] * w[1] + K[2] * w[2]) / (safe * safe)
    for a in range(3):
        w[a] = (w[a] - K[a] * kdot) * amp
    return w, K


def _field(N, seed, dtype):
    """u[x3][x2][x1][a], unit rms."""
    w, _ = _solenoidal(N, seed, dtype)
    u = torch.empty((N, N, N, 3), device=DEV, dtype=dtype)
    for a in range(3):
        u[..., a] = torch.fft.irfftn(w[a], s=(N, N, N))
        w[a] = None
    ms = 0.0
    for z in range(0, N, 64):
        ms += float(u[z:z + 64].double().square().sum())
    u *= 1.0 / math.sqrt(ms / u.numel())
    return u


def _spectrum(case, seed):
    """The half spectrum [k2][k3][k1][a] of a velocity of unit rms, or of its vorticity."""
    N = case["N"]
    w, K = _solenoidal(N, seed, torch.float64)
    # Parseval: the modes with 0 < k1 < N/2 stand for two
    twice = torch.full((1, 1, N // 2 + 1), 2.0, device=DEV, dtype=torch.float64)
    twice[..., 0] = 1.0
    twice[..., N // 2] = 1.0
    ms = sum(float((v.abs().square() * twice).sum()) for v in w) / 3.0
    s = 1.0 / math.sqrt(ms)
    if case["kind"] == "vorticity":  # i k x u
        w = [1j * (K[(a + 1) % 3] * w[(a + 2) % 3] - K[(a + 2) % 3] * w[(a + 1) % 3]) for a in range(3)]
    dtype = torch.complex128 if case["spec"] == "c128" else torch.complex64
    out = torch.empty((N, N, N // 2 + 1, 3), device=DEV, dtype=dtype)
    for a in range(3):
        out[..., a] = (w[a] * s).transpose(0, 1)
        w[a] = None
    return out


def _positions(n, seed):
    g = _gen(seed, 1)
    X = torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64)
    X *= L
    k = n // 16  # tracers that have crossed a periodic face
    X[:k] += L * torch.randint(-1, 2, (k, 3), generator=g, device=DEV).double()
    return X[torch.randperm(n, generator=g, device=DEV)] if n < 1 << 20 else X


def _axes(n, seed):
    p = torch.randn((n, 3), generator=_gen(seed, 2), device=DEV, dtype=torch.float64)
    return p / p.norm(dim=1, keepdim=True)


def _params(seed):
    """Initial weights of the network, with a small output layer."""
    g = torch.Generator()
    g.manual_seed(int(seed))
    w1 = torch.randn((HIDDEN, FEATURES), generator=g) / math.sqrt(FEATURES)
    w2 = torch.randn((HIDDEN, HIDDEN), generator=g) / math.sqrt(HIDDEN)
    w3 = torch.randn((3, HIDDEN), generator=g) * (2e-3 / math.sqrt(HIDDEN))
    b = [0.05 * torch.randn((k,), generator=g) for k in (HIDDEN, HIDDEN)]
    return torch.cat([w1.reshape(-1), b[0], w2.reshape(-1), b[1], w3.reshape(-1), torch.zeros(3)]).numpy()


def _inputs(case, seed):
    """Everything that is drawn: field or spectrum, positions, axes or velocities."""
    do, N = case["do"], case["N"]
    d = {}
    if do == "loop":
        d["spec"] = _spectrum(case, seed)
    else:
        dtype = torch.float64 if case["storage"] == "f64" else torch.float32
        d["u"] = _field(N, seed, dtype)
        if do == "next":
            d["u2"] = _field(N, seed + 7919, dtype)
    d["X"] = _positions(case["np"], seed)
    if case["type"] == "axes":
        d["p"] = _axes(case["np"], seed)
    if case["type"] == "inertia":
        d["V"] = torch.randn((case["np"], 3), generator=_gen(seed, 3), device=DEV, dtype=torch.float64)
    return d


def prepare(case, seed):
    do, n = case["do"], case["np"]
    s = _inputs(case, seed)
    ctx = ptk.Context(0)
    family = ptk.LAGRANGE if case["family"] == "lagrange" else ptk.SPLINE
    k = (family, case["I"], case["m"], STORE[case["storage"]])
    if do == "loop":
        ctx.set_field_spectral(s["spec"], *k, kind=_kind(case))
    else:
        ctx.set_field(s.pop("u"), *k)
    s.update(ctx=ctx, case=case, k=k)
    vel = torch.float64 if case["storage"] == "f64" else torch.float32
    depth = ORDER.get(case["scheme"], 0)
    if do == "noalloc":
        s["out"] = torch.empty((n, 3), dtype=vel, device=DEV)
    if do == "advance":
        s["hist"] = torch.zeros((depth, n, 3), dtype=vel, device=DEV) if depth else None
        s["hl"] = 0
    if do in ("resident", "loop", "next"):
        ctx.particles_load(s["X"], hist_depth=depth if do == "resident" else 0)
        if case["type"] == "axes":
            ctx.particles_set_orientation(s["p"], SHAPE)
        if case["type"] == "inertia":
            ctx.particles_set_inertia(s["V"], TAU)
        s["hist"] = torch.zeros((depth, n, 3), dtype=vel, device=DEV) if do == "resident" and depth else None
    if do in ("advance", "resident", "loop", "next"):
        s["g"] = torch.empty((n, 3, 3), dtype=vel, device=DEV) if case["grad"] else None
    if do in ("learned", "batch"):
        ctx.learned_set_params(_params(seed))
    if do == "batch":
        s["feat"], s["target"] = ctx.learned_make_pairs(s["X"])
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return s


def _kind(case):
    return ptk.SPEC_VORTICITY if case["kind"] == "vorticity" else ptk.SPEC_VELOCITY


def run(s):
    case, ctx, X = s["case"], s["ctx"], s["X"]
    do = case["do"]
    vel = torch.float64 if case["storage"] == "f64" else torch.float32
    if do == "interp":
        return ctx.interpolate_gradient(X, out_dtype=vel) if case["grad"] else ctx.interpolate(X, out_dtype=vel)
    if do == "noalloc":
        return ctx.interpolate_noalloc(X, s["out"])
    if do == "learned":
        out, rms, fell_back = ctx.interpolate_learned(X, audit_frac=1e-3, tol_rel_rms=10.0)
        return out, rms, fell_back
    if do == "batch":
        return ctx.learned_loss_grad(s["feat"], s["target"])
    scheme = SCHEMES[case["scheme"]]
    if do == "advance":
        s["hl"] = ctx.advance(X, scheme, case["dt"], case["nsteps"], hist=s["hist"], hist_len=s["hl"], grad_out=s["g"])
        return {"X": X, "hist": None if s["hist"] is None else s["hist"][:s["hl"]], "grad": s["g"]}
    if do == "loop":
        ctx.set_field_spectral(s["spec"], *s["k"], kind=_kind(case))
        ctx.particles_advance(ptk.HEUN, case["dt"], 1, grad_out=s["g"])
    elif do == "next":
        ctx.set_field_next(s["u2"])
        ctx.particles_step_next_field(case["dt"], grad_out=s["g"])
    else:
        ctx.particles_advance(scheme, case["dt"], case["nsteps"], grad_out=s["g"])
    hl = ctx.particles_store(X, hist=s.get("hist"))
    out = {"X": X, "hist": s["hist"][:hl] if hl else None, "grad": s["g"]}
    if case["type"] == "axes":
        ctx.particles_get_orientation(s["p"])
        out["p"] = s["p"]
    if case["type"] == "inertia":
        ctx.particles_get_inertia(s["V"])
        out["V"] = s["V"]
    return out


def work(case):
    n, I, N = case["np"], case["I"], case["N"]
    if case["do"] == "batch":
        mac = HIDDEN * FEATURES + HIDDEN * HIDDEN + 3 * HIDDEN
        return {"bytes": n * (2 * PITCH + 12) + 8 * 41987, "flops": 6.0 * mac * n}
    v = 8 if case["storage"] == "f64" else 4
    node = NODE_BYTES[case["storage"]]
    field = min(N ** 3, n * I ** 3) * node  # each node that some particle reads, once
    evals = 2 if case["scheme"] == "heun" else 1
    pts = n * 24 + n * 3 * v
    value, grad = 6.0 * (I ** 3 + I ** 2 + I), 12.0 * (I ** 3 + I ** 2 + I)
    g = n * 9 * v if case["grad"] else 0
    if case["do"] in ("interp", "noalloc"):
        return {"bytes": field + pts + g, "flops": n * (grad if case["grad"] else value)}
    if case["do"] == "learned":
        return {"bytes": field + pts, "flops": 2.0 * n * (HIDDEN * FEATURES + HIDDEN * HIDDEN + 3 * HIDDEN + 3 * 84)}
    if case["do"] in ("loop", "next"):
        evals, steps = 2, 1
    else:
        steps = case["nsteps"]
    state = 48 * n  # positions in and out; axes or velocities likewise
    if case["type"] != "tracers":
        state += 48 * n
    hist = 2 * ORDER.get(case["scheme"], 0) * 3 * v * n if case["do"] in ("advance", "resident") else 0
    total = steps * evals * field + state + hist + g
    per = grad if case["type"] == "axes" else value
    flops = n * (steps * evals * per + (grad - value if case["grad"] else 0))
    if case["do"] == "loop":
        cplx = 16 if case["spec"] == "c128" else 8
        total += 3 * N * N * (N // 2 + 1) * cplx + N ** 3 * node
        flops += 3 * 2.5 * N ** 3 * 3 * math.log2(N)
    if case["do"] == "next":
        total += N ** 3 * (3 * v + node)
    return {"bytes": float(total), "flops": float(flops)}


# ---------------------------------------------------------------- the same in 64 bits, in plain torch

def _mul(a, b):
    out = [Fraction(0)] * (len(a) + len(b) - 1)
    for i, x in enumerate(a):
        for j, y in enumerate(b):
            out[i + j] += x * y
    return out


def _diff(p, k):
    for _ in range(k):
        p = [i * p[i] for i in range(1, len(p))] or [Fraction(0)]
    return p


def _at(p, x):
    return sum((c * Fraction(x) ** i for i, c in enumerate(p)), Fraction(0))


def _lagrange(nodes, j):
    p = [Fraction(1)]
    for k in nodes:
        if k != j:
            p = _mul(p, [Fraction(-k, j - k), Fraction(1, j - k)])
    return p


def _polynomials(family, I, m):
    """beta_j in ascending powers of t, node offsets 1 - I/2 .. I/2."""
    n = I // 2 - 1
    nodes = list(range(-n, n + 2))
    if family == "lagrange":
        return [_lagrange(nodes, j) for j in nodes]
    left, right = nodes[:-1], nodes[1:]
    extra = list(range(-(n - m), 0)) + list(range(2, n - m + 2))
    deg = I - 1
    unit = [[Fraction(0)] * i + [Fraction(1)] for i in range(deg + 1)]
    conds = [(x, k) for k in range(m + 1) for x in (0, 1)] + [(x, 0) for x in extra]
    rows = [[_at(_diff(e, k), x) for e in unit] for x, k in conds]
    out = []
    for j in nodes:
        rhs = []
        for x, k in conds:
            if k == 0:
                rhs.append(Fraction(int(j == x)))
            else:
                own = left if x == 0 else right
                rhs.append(_at(_diff(_lagrange(own, j), k), x) if j in own else Fraction(0))
        M = [list(r) + [b] for r, b in zip(rows, rhs)]
        for col in range(deg + 1):  # Gauss-Jordan in exact rationals
            piv = next(r for r in range(col, deg + 1) if M[r][col] != 0)
            M[col], M[piv] = M[piv], M[col]
            M[col] = [v / M[col][col] for v in M[col]]
            for r in range(deg + 1):
                if r != col and M[r][col] != 0:
                    M[r] = [a - M[r][col] * b for a, b in zip(M[r], M[col])]
        out.append([M[r][deg + 1] for r in range(deg + 1)])
    return out


def _horner(polys, t):
    w = torch.empty(t.shape + (len(polys),), dtype=torch.float64, device=t.device)
    for j, p in enumerate(polys):
        acc = torch.full_like(t, float(p[-1]))
        for c in reversed(p[:-1]):
            acc = acc * t + float(c)
        w[..., j] = acc
    return w


def _cells(X, N):
    s = torch.remainder(X, L) * (N / L)
    c = s.floor()
    t = s - c
    return c.long() % N, t


def _weighted_sum(u, X, kernel, grad, chunk=1 << 20):
    """u(X) and its gradient by the triple sum, FP64."""
    N = u.shape[0]
    flat = u.reshape(-1, 3)
    P = _polynomials(*kernel)
    I = len(P)
    D = [_diff(p, 1) for p in P]
    val = torch.empty((X.shape[0], 3), dtype=torch.float64, device=X.device)
    out = torch.empty((X.shape[0], 3, 3), dtype=torch.float64, device=X.device) if grad else None
    off = torch.arange(1 - I // 2, I // 2 + 1, device=X.device)
    for b in range(0, X.shape[0], chunk):
        c, t = _cells(X[b:b + chunk], N)
        w = _horner(P, t)
        d = _horner(D, t) if grad else None
        ix = [(c[:, q, None] + off) % N for q in range(3)]
        acc = [torch.zeros((c.shape[0], 3), dtype=torch.float64, device=X.device) for _ in range(4 if grad else 1)]
        for k3 in range(I):
            for k2 in range(I):
                row = (ix[2][:, k3] * N + ix[1][:, k2]) * N
                v = flat[row[:, None] + ix[0]].double()
                s = (v * w[:, 0, :, None]).sum(1)
                w2, w3 = w[:, 1, k2, None], w[:, 2, k3, None]
                acc[0] += s * (w2 * w3)
                if grad:
                    acc[1] += (v * d[:, 0, :, None]).sum(1) * (w2 * w3)
                    acc[2] += s * (d[:, 1, k2, None] * w3)
                    acc[3] += s * (w2 * d[:, 2, k3, None])
        val[b:b + chunk] = acc[0]
        if grad:
            out[b:b + chunk] = torch.stack(acc[1:], dim=2) * (N / L)
    return val, out


def _grid_of(case, spec):
    """The velocity on the grid of a half spectrum [k2][k3][k1][a], FP64."""
    N = case["N"]
    K = _wave_numbers(N, torch.float64)
    w = [spec[..., a].transpose(0, 1).to(torch.complex128) for a in range(3)]
    if case["kind"] == "vorticity":
        kk = K[0] * K[0] + K[1] * K[1] + K[2] * K[2]
        keep = (kk > 0) & (K[0].abs() < N / 2) & (K[1].abs() < N / 2) & (K[2].abs() < N / 2)
        f = torch.where(keep, 1.0 / kk.clamp(min=1.0), torch.zeros_like(kk))
        w = [1j * (K[(a + 1) % 3] * w[(a + 2) % 3] - K[(a + 2) % 3] * w[(a + 1) % 3]) * f for a in range(3)]
    u = torch.empty((N, N, N, 3), device=DEV, dtype=torch.float64)
    for a in range(3):
        u[..., a] = torch.fft.irfftn(w[a], s=(N, N, N), norm="forward")
        w[a] = None
    return u


def _jeffery(G, p):
    S, W = 0.5 * (G + G.transpose(1, 2)), 0.5 * (G - G.transpose(1, 2))
    Sp, Wp = (S * p[:, None, :]).sum(2), (W * p[:, None, :]).sum(2)
    return Wp + SHAPE * (Sp - (p * Sp).sum(1, keepdim=True) * p)


def _step(case, d, fields):
    """One prepared state after its steps: outputs of run() in FP64."""
    kernel = (case["family"], case["I"], case["m"])
    X, dt, kind = d["X"], case["dt"], case["type"]
    q = d.get("p", d.get("V"))
    depth = ORDER.get(case["scheme"], 0) if case["do"] in ("advance", "resident") else 0
    steps = case["nsteps"] if case["do"] in ("advance", "resident") else 1
    scheme = case["scheme"] if case["do"] in ("advance", "resident") else "heun"
    grad, hist, hx, hq = None, [], [], []

    def rates(u, X, q, want):
        v, g = _weighted_sum(u, X, kernel, want or kind == "axes")
        if kind == "axes":
            return v, v, _jeffery(g, q), g
        if kind == "inertia":
            return v, q, (v - q) / TAU, g
        return v, v, None, g

    for k in range(steps):
        v, rx, rq, g = rates(fields[0], X, q, case["grad"] and k == steps - 1)
        if case["grad"] and k == steps - 1:
            grad = g
        if scheme == "heun":
            q1 = None if q is None else q + dt * rq
            _, rx2, rq2, _ = rates(fields[-1], X + dt * rx, q1, False)
            X = X + 0.5 * dt * (rx + rx2)
            q = None if q is None else q + 0.5 * dt * (rq + rq2)
        else:
            b = AB[min(depth, len(hx) + 1)] if depth else AB[1]
            X = X + dt * sum(c * r for c, r in zip(b, [rx] + hx))
            q = None if q is None else q + dt * sum(c * r for c, r in zip(b, [rq] + hq))
            if depth:
                hist, hx, hq = ([v] + hist)[:depth], ([rx] + hx)[:depth], ([rq] + hq)[:depth]
        if kind == "axes":
            q = q / q.norm(dim=1, keepdim=True)
    out = {"X": X, "hist": torch.stack(hist) if hist else None, "grad": grad}
    if kind == "axes":
        out["p"] = q
    if kind == "inertia":
        out["V"] = q
    return out


def _network(params, x):
    o, w = 0, []
    for shape in ((HIDDEN, FEATURES), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (3, HIDDEN), (3,)):
        k = math.prod(shape)
        w.append(params[o:o + k].view(shape))
        o += k
    h = torch.nn.functional.silu(x @ w[0].t() + w[1])
    h = torch.nn.functional.silu(h @ w[2].t() + w[3])
    return h @ w[4].t() + w[5]


def _features(u, X):
    """Stencil of the four-point kernel and the offsets, as the network takes them (rounded to BF16)."""
    N = u.shape[0]
    c, t = _cells(X, N)
    off = torch.arange(-1, 3, device=X.device)
    ix = [(c[:, q, None] + off) % N for q in range(3)]
    rows = (ix[2][:, :, None, None] * N + ix[1][:, None, :, None]) * N + ix[0][:, None, None, :]
    f = torch.cat([u.reshape(-1, 3)[rows.reshape(X.shape[0], -1)].reshape(X.shape[0], -1).float(), t.float()], dim=1)
    return f.bfloat16().double()


def exact(case, seed):
    do = case["do"]
    d = _inputs(case, seed)
    kernel = (case["family"], case["I"], case["m"])
    if do in ("interp", "noalloc"):
        v, g = _weighted_sum(d["u"], d["X"], kernel, case["grad"])
        return (v, g) if case["grad"] else v
    if do == "learned":
        params = torch.from_numpy(_params(seed)).to(DEV).double()
        out = torch.empty_like(d["X"])
        for b in range(0, d["X"].shape[0], 1 << 19):
            X = d["X"][b:b + (1 << 19)]
            out[b:b + (1 << 19)] = _weighted_sum(d["u"], X, ("lagrange", 4, 0), False)[0] + _network(params, _features(d["u"], X))
        return out, None, 0
    if do == "batch":
        params = torch.from_numpy(_params(seed)).to(DEV).double().requires_grad_(True)
        target = _weighted_sum(d["u"], d["X"], kernel, False)[0] - _weighted_sum(d["u"], d["X"], ("lagrange", 4, 0), False)[0]
        loss = (_network(params, _features(d["u"], d["X"])) - target).square().mean()
        loss.backward()
        return loss.detach().reshape(1), params.grad
    fields = [_grid_of(case, d["spec"])] if do == "loop" else [d["u"], d["u2"]] if do == "next" else [d["u"]]
    return _step(case, d, fields)
