"""Particles evaluated straight from the field (few of them for the grid)
against the same particles in calls large enough to be binned and swept: the
two kernels add in the same order, so results agree bit for bit.  The oracle
tests run small calls; through this equality they hold for large ones too."""
import numpy as np
import pytest
import torch

from oracle import geometry, kernels as K

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
L = geometry.L


@pytest.fixture(scope="module")
def ptk(lib):
    return lib


def field(N, seed, dtype=torch.float32):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn((N, N, N, 3), generator=g, device=DEV, dtype=dtype) + 0.5


def positions(N, n, seed):
    """Uniform over three periods, the first ones on nodes, faces and just below them."""
    rng = np.random.default_rng(seed)
    X = rng.uniform(-L, 2 * L, (n, 3))
    e = np.array([0.0, -0.0, L, -L, np.nextafter(L, 0), np.nextafter(0, -1), 12 * L / N, np.nextafter(12 * L / N, 0),
                  (N - 1) * L / N, 5 * L / N, np.pi])
    X[:200] = rng.choice(e, (200, 3))
    return torch.from_numpy(X).to(DEV)


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("fam,I,m", [(K.LAGRANGE, 4, 0), (K.SPLINE, 6, 1), (K.SPLINE, 8, 2)])
@pytest.mark.parametrize("N,n", [(67, 500_000), (9, 300_000)])
def test_small_call_equals_its_rows_of_a_large_one(ptk, storage, fam, I, m, N, n):
    print(f"[direct] {storage} I={I} N={N} n={n}", flush=True)
    ctx = ptk.Context(0)
    f64 = storage == "f64"
    ctx.set_field(field(N, N + I, torch.float64 if f64 else torch.float32), fam, I, m,
                  storage={"f64": ptk.F64, "f32": ptk.F32, "bf16": ptk.BF16, "f16": ptk.F16}[storage])
    X = positions(N, n, I)
    for out in (torch.float32, torch.float64):
        v = ctx.interpolate(X, out_dtype=out)
        u, g = ctx.interpolate_gradient(X, out_dtype=out)
        for k in (1, 17, 1003):
            assert torch.equal(ctx.interpolate(X[:k].contiguous(), out_dtype=out), v[:k])
            us, gs = ctx.interpolate_gradient(X[:k].contiguous(), out_dtype=out)
            assert torch.equal(us, u[:k]) and torch.equal(gs, g[:k])
    ctx.close()


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("scheme", ["EULER", "HEUN", "AB2", "AB4"])
def test_small_advance_equals_its_rows_of_a_large_one(ptk, storage, scheme):
    """Six steps with the last one's gradient; more steps than one launch takes
    for the small call alone."""
    N, n, k = 64, 500_000, 777
    print(f"[direct steps] {storage} {scheme}", flush=True)
    dt = torch.float64 if storage == "f64" else torch.float32
    ctx = ptk.Context(0)
    ctx.set_field(field(N, 3, dt), K.SPLINE, 8, 2, storage=ptk.F64 if storage == "f64" else ptk.F32)
    sch = getattr(ptk, scheme)
    depth = ptk.AB_ORDER.get(sch, 0)

    def run(X, calls, grad=True):
        n = X.shape[0]
        hist = torch.zeros((depth, n, 3), dtype=dt, device=DEV) if depth else None
        g, hl = torch.zeros((n, 3, 3), dtype=dt, device=DEV) if grad else None, 0
        for c in calls:
            hl = ctx.advance(X, sch, 2e-3, c, hist=hist, hist_len=hl, grad_out=g)
        return X, g, hl, hist

    X0 = positions(N, n, 5)
    a = run(X0.clone(), [1, 5])
    b = run(X0[:k].clone(), [1, 5])
    assert torch.equal(a[0][:k], b[0]) and torch.equal(a[1][:k], b[1]) and a[2] == b[2]
    if depth:
        assert torch.equal(a[3][:, :k], b[3])
    # (no gradient: the steps that return one take their velocity from its kernel)
    c, d = run(X0[:k].clone(), [130], False), run(X0[:k].clone(), [60, 70], False)
    assert torch.equal(c[0], d[0])
    ctx.close()


@pytest.mark.parametrize("kind", ["tracers", "axes", "inertia"])
@pytest.mark.parametrize("scheme", ["HEUN", "AB3"])
@pytest.mark.parametrize("order", [(4, 8, 4), (8, 4, 8)])
def test_resident_state_across_kernels_of_other_reach(ptk, kind, scheme, order):
    """150 000 particles on 64^3 are swept with I = 8 and read directly with
    I = 4: a resident run that changes the kernel goes through both, and agrees
    with one particle set of a size that is always read directly."""
    N, n, k = 64, 150_000, 300
    print(f"[direct resident] {kind} {scheme} {order}", flush=True)
    u = field(N, 8)
    rng = np.random.default_rng(4)
    p = rng.standard_normal((n, 3))
    p = torch.from_numpy(p / np.linalg.norm(p, axis=1, keepdims=True)).to(DEV)
    X0 = positions(N, n, 6)
    sch = getattr(ptk, scheme)
    depth = ptk.AB_ORDER.get(sch, 0)

    def run(X, p):
        ctx = ptk.Context(0)
        g = torch.zeros((X.shape[0], 3, 3), dtype=torch.float32, device=DEV)
        hist = torch.zeros((depth, X.shape[0], 3), dtype=torch.float32, device=DEV) if depth else None
        for e, I in enumerate(order):
            ctx.set_field(u, K.LAGRANGE if I == 4 else K.SPLINE, I, 0 if I == 4 else 2, storage=ptk.F32)
            if e == 0:
                ctx.particles_load(X, hist_depth=depth)
                if kind == "axes":
                    ctx.particles_set_orientation(p, 0.7)
                elif kind == "inertia":
                    ctx.particles_set_inertia(p, 0.2)
            ctx.particles_advance(sch, 2e-3, 2, grad_out=g)
        hl = ctx.particles_store(X, hist=hist)
        ph, vh = (torch.zeros((depth, X.shape[0], 3), dtype=torch.float64, device=DEV) for _ in range(2))
        if kind == "axes":
            ctx.particles_get_orientation(p, hist=ph)
        elif kind == "inertia":
            ctx.particles_get_inertia(p, v_hist=vh, r_hist=ph)
        ctx.close()
        return X, g, p, hl, hist, ph, vh

    a, b = run(X0.clone(), p.clone()), run(X0[:k].clone(), p[:k].clone())
    assert torch.equal(a[0][:k], b[0]) and torch.equal(a[1][:k], b[1]) and torch.equal(a[2][:k], b[2])
    assert a[3] == b[3]
    if depth:
        assert torch.equal(a[4][:, :k], b[4]) and torch.equal(a[5][:, :k], b[5]) and torch.equal(a[6][:, :k], b[6])


def test_binning_of_a_direct_call(ptk):
    """ptk_get_binning after a call that did not sort: the stable order, at every
    call and after resident particles moved in between."""
    N, n = 32, 2003
    print("[direct binning]", flush=True)
    ctx = ptk.Context(0)
    ctx.set_field(field(N, 1), K.SPLINE, 8, 2, storage=ptk.F32)
    X = positions(N, n, 2)
    ctx.particles_load(X[:100].contiguous())
    ctx.interpolate(X)
    keys = geometry.bin_keys(X.cpu().numpy(), N, 12, 5)
    for _ in range(2):
        perm, off, T, W = ctx.binning()
        assert np.array_equal(perm.cpu().numpy().astype(np.int64), geometry.stable_order(keys))
        assert np.array_equal(off.cpu().numpy().astype(np.int64),
                              geometry.offsets_from_keys(keys, geometry.n_bins(N, T, W)))
        ctx.particles_advance(ptk.HEUN, 1e-3, 1)
    ctx.close()
