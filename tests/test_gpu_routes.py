"""The ways a call's particles are evaluated (straight from the field, the same
in bin order, the binned sweep), where a call's size or shape changes them.
PTK_TEST_ROUTE, read when a context is made, takes the choice from the rule.

The kernels add in the same order, so the routes agree bit for bit; the oracle
tests' calls are small and mostly read directly, and through this equality they
hold for the sweep too.  (Every case forces its routes: what the rule would
choose plays no part.)"""
import numpy as np
import pytest
import torch

from oracle import geometry, kernels as K

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
L = geometry.L


ROUTES = ("direct", "sorted", "sweep")
KERNELS = [(K.LAGRANGE, 4, 0), (K.SPLINE, 6, 1), (K.SPLINE, 8, 2)]


@pytest.fixture(scope="module")
def ptk(lib):
    return lib


def field(N, seed, storage):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn((N, N, N, 3), generator=g, device=DEV,
                       dtype=torch.float64 if storage == "f64" else torch.float32) + 0.5


def positions(N, n, seed):
    """Uniform over three periods, the first ones on nodes, faces and just below them."""
    rng = np.random.default_rng(seed)
    X = rng.uniform(-L, 2 * L, (n, 3))
    e = np.array([0.0, -0.0, L, -L, np.nextafter(L, 0), np.nextafter(0, -1), 12 * L / N, np.nextafter(12 * L / N, 0),
                  (N - 1) * L / N, 5 * L / N, np.pi])
    X[:200] = rng.choice(e, (min(n, 200), 3))
    return torch.from_numpy(X).to(DEV)


def same(a, b):
    """Bit for bit, NaN for NaN."""
    return torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.nan_to_num(a), torch.nan_to_num(b))


def evaluations(ctx, X, out_dtypes=(torch.float32, torch.float64)):
    res = []
    for out in out_dtypes:
        res += [ctx.interpolate(X, out_dtype=out), *ctx.interpolate_gradient(X, out_dtype=out),
                ctx.interpolate_gradient(X, out_dtype=out, with_value=False)[1]]
        res.append(ctx.interpolate_noalloc(X, torch.full_like(res[-4], float("nan"))))
    return res


def context(ptk, monkeypatch, route):
    monkeypatch.setenv("PTK_TEST_ROUTE", route)
    ctx = ptk.Context(0)
    monkeypatch.delenv("PTK_TEST_ROUTE")
    return ctx


def test_direct_calls_of_more_particles_than_a_launch_takes(ptk, monkeypatch):
    """2^28 + 21 particles (16 work-items each: more than 2^32) read directly: 256
    copies of 2^20 positions and a few more, one call and one step, against the
    call and the step of the 2^20."""
    N, m = 8, 1 << 20
    n = 256 * m + 21
    print(f"[routes] {n} particles directly", flush=True)
    g = torch.Generator(device=DEV).manual_seed(1)
    u = torch.randn((N, N, N, 3), generator=g, device=DEV)
    base = torch.rand((m, 3), generator=g, device=DEV, dtype=torch.float64) * L
    ctx = context(ptk, monkeypatch, "direct")
    ctx.set_field(u, ptk.LAGRANGE, 4, 0, storage=ptk.F32)
    X = torch.empty((n, 3), dtype=torch.float64, device=DEV)
    X[:256 * m].view(256, m, 3).copy_(base)
    X[256 * m:] = base[:21]

    def same(got, ref):
        assert torch.equal(got[:256 * m].view(256, m, 3), ref.expand(256, m, 3))
        assert torch.equal(got[256 * m:], ref[:21])

    out = torch.full((n, 3), float("nan"), device=DEV)
    ctx.interpolate(X, out=out)
    same(out, ctx.interpolate(base))
    del out
    ctx.advance(X, ptk.EULER, 1e-2, 1)
    ctx.advance(base, ptk.EULER, 1e-2, 1)
    same(X, base)
    ctx.close()
    del X
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33])
def test_direct_steps_at_the_edges_of_a_block(ptk, monkeypatch, n):
    """70 AB3 steps (two launches) in place, history with them, against the same
    particles among 64: a block takes 16 particles, and what its last lanes have
    no particle for may not touch the others'."""
    print(f"[routes] {n} particles, 70 steps", flush=True)
    g = torch.Generator(device=DEV).manual_seed(n)
    u = torch.randn((16, 16, 16, 3), generator=g, device=DEV)
    X0 = torch.rand((64, 3), generator=g, device=DEV, dtype=torch.float64) * L
    ctx = context(ptk, monkeypatch, "direct")
    ctx.set_field(u, ptk.SPLINE, 6, 1, storage=ptk.F32)

    def run(X):
        h = torch.zeros((3, X.shape[0], 3), device=DEV)
        gr = torch.zeros((X.shape[0], 3, 3), device=DEV)
        assert ctx.advance(X, ptk.AB3, 1e-3, 70, hist=h, grad_out=gr) == 3
        return X, h, gr

    a, b = run(X0.clone()), run(X0[:n].clone())
    assert torch.equal(a[0][:n], b[0]) and torch.equal(a[1][:, :n], b[1]) and torch.equal(a[2][:n], b[2])
    ctx.close()


@pytest.mark.parametrize("kind,one_shot", [("tracers", False), ("tracers", True), ("axes", False), ("inertia", False)])
@pytest.mark.parametrize("scheme", ["EULER", "HEUN", "AB3"])
def test_steps_in_bin_order_keep_it(ptk, monkeypatch, kind, scheme, one_shot):
    """Steps evaluated in bin order sort the state again after every eight, with
    the sweep's results bit for bit (which re-bins after each, but for a
    one-shot call's last)."""
    print(f"[routes] bin order kept: {kind} {scheme} one_shot={one_shot}", flush=True)
    N, n, steps = 24, 9001, 27
    g = torch.Generator(device=DEV).manual_seed(3)
    u = torch.randn((N, N, N, 3), generator=g, device=DEV)
    X0 = (torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64) * 3 - 1) * L
    p0 = torch.nn.functional.normalize(torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64))
    sch = getattr(ptk, scheme)
    depth = ptk.AB_ORDER.get(sch, 0)

    def run(route):
        ctx = context(ptk, monkeypatch, route)
        ctx.set_field(u, ptk.SPLINE, 8, 2, storage=ptk.F32)
        X, p = X0.clone(), p0.clone()
        h = torch.zeros((depth, n, 3), device=DEV) if depth else None
        ph, vh = (torch.zeros((depth, n, 3), device=DEV, dtype=torch.float64) for _ in range(2))
        gr = torch.zeros((n, 3, 3), device=DEV)
        ctx.timing(True)
        if one_shot:
            ctx.advance(X, sch, 2e-2, steps, hist=h, grad_out=gr)
        else:
            ctx.particles_load(X, hist_depth=depth)
            if kind == "axes":
                ctx.particles_set_orientation(p, 0.7)
            elif kind == "inertia":
                ctx.particles_set_inertia(p, 0.2)
            ctx.particles_advance(sch, 2e-2, 5)
            ctx.particles_advance(sch, 2e-2, steps - 5, grad_out=gr)
            ctx.particles_store(X, hist=h)
            if kind == "axes":
                ctx.particles_get_orientation(p, hist=ph)
            elif kind == "inertia":
                ctx.particles_get_inertia(p, v_hist=vh, r_hist=ph)
        sorts = ctx.timing_read()["sort"][1]
        ctx.close()
        return sorts, [X, p, gr, ph, vh] + ([h] if depth else [])

    sorts, a = run("sorted")
    assert sorts == 1 + (steps - 1) // 8
    swept, b = run("sweep")
    assert swept == 1 + steps - (1 if one_shot else 0) + (steps if scheme == "HEUN" else 0)  # (the predictor's bins too)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    none, d = run("direct")
    assert none == 0
    for x, y in zip(a, d):
        assert torch.equal(x, y)


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("fam,I,m", KERNELS)
@pytest.mark.parametrize("N", [8, 9, 12, 13, 67])
def test_routes_agree(ptk, monkeypatch, storage, fam, I, m, N):
    """Grids below, at and beyond a tile's edge; a particle, a ragged count and
    (swept, with several chunks in every window) a crowd."""
    print(f"[routes] {storage} I={I} N={N}", flush=True)
    u = field(N, N + I, storage)
    for n in (1, 3001, 40_000):
        X = positions(N, n, n + I)
        ref = None
        for route in ROUTES:
            ctx = context(ptk, monkeypatch, route)
            ctx.set_field(u, fam, I, m, storage=getattr(ptk, storage.upper()))
            got = evaluations(ctx, X)
            ctx.close()
            ref = ref or got
            for a, b in zip(got, ref):
                assert torch.equal(a, b), (n, route)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("fam,I,m", KERNELS)
def test_routes_agree_on_infinities_and_nan(ptk, monkeypatch, storage, fam, I, m):
    print(f"[routes] non-finite nodes, {storage} I={I}", flush=True)
    N, n = 29, 20_000
    u = field(N, I, storage)
    rng = np.random.default_rng(I)
    for bad in (float("inf"), float("-inf"), float("nan")):
        i = torch.from_numpy(rng.integers(0, N, (4, 3))).to(DEV)
        u[i[:, 0], i[:, 1], i[:, 2], int(rng.integers(0, 3))] = bad
    X = positions(N, n, I)
    ref = None
    for route in ROUTES:
        ctx = context(ptk, monkeypatch, route)
        ctx.set_field(u, fam, I, m, storage=getattr(ptk, storage.upper()))
        got = evaluations(ctx, X, (torch.float64,))
        ctx.close()
        ref = ref or got
        for a, b in zip(got, ref):
            assert same(a, b), route
    assert bool(torch.isnan(ref[0]).any()) and bool(torch.isfinite(ref[0]).any())


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("fam,I,m", KERNELS)
def test_crowded_windows_beside_empty_ones(ptk, monkeypatch, storage, fam, I, m):
    """130^3: segments of three windows of five layers (the last of two), 160
    particles a chunk.  Windows with nothing, one particle, and counts at the
    edges of one, two and many chunks, first, in the middle and last in their
    segment."""
    print(f"[routes] crowded windows, {storage} I={I}", flush=True)
    N = 130
    u = field(N, I, storage)
    rng = np.random.default_rng(I)
    counts = [0, 0, 1000, 161, 0, 0, 0, 320, 0, 159, 160, 161, 0, 0, 0, 1, 0, 321, 2000, 2000, 1, 0, 1, 0, 481, 1999]
    assert len(counts) == -(-N // 5)
    rows = []
    for column in ((0, 0), (0, 10), (7, 3), (10, 10)):  # the last columns are ten cells wide
        for w, c in enumerate(counts if column != (7, 3) else counts[::-1]):
            lo = np.array([12 * column[0], 12 * column[1], 5 * w])
            hi = np.minimum(lo + [12, 12, 5], N)
            rows.append(rng.uniform(lo, hi, (c, 3)))
    X = np.concatenate(rows)
    X = torch.from_numpy(rng.permutation(X) * (L / N)).to(DEV)
    ref = None
    for route in ROUTES:
        ctx = context(ptk, monkeypatch, route)
        ctx.set_field(u, fam, I, m, storage=getattr(ptk, storage.upper()))
        got = evaluations(ctx, X, (torch.float32,))
        ctx.close()
        ref = ref or got
        for a, b in zip(got, ref):
            assert torch.equal(a, b), route


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("N,n", [(8, 0), (16, 1), (16, 2047), (16, 2048), (16, 2049), (24, 70_001), (60, 500_001)])
def test_permutation_on_every_route(ptk, monkeypatch, route, N, n):
    """The recorded binning is the stable order of the keys, however often it is
    asked for and whatever a resident state does in between; single tiles,
    their edges, one and two digit passes."""
    print(f"[routes] binning, {route} N={N} n={n}", flush=True)
    ctx = context(ptk, monkeypatch, route)
    ctx.set_field(field(N, 1, "f32"), ptk.LAGRANGE, 4, 0, storage=ptk.F32)
    rng = np.random.default_rng(n)
    cells = rng.integers(0, N, (n, 3))
    X = torch.from_numpy((cells + 0.5) * (L / N)).to(DEV)
    ctx.particles_load(positions(N, 500, 2), hist_depth=2)
    ctx.interpolate(X)
    for _ in range(2):
        perm, off, T, W = ctx.binning()
        nt, nw = -(-N // T), -(-N // W)
        key = ((cells[:, 1] // T) * nt + cells[:, 0] // T) * nw + cells[:, 2] // W
        np.testing.assert_array_equal(perm.cpu().numpy(), np.argsort(key, kind="stable"))
        np.testing.assert_array_equal(off.cpu().numpy()[1:], np.cumsum(np.bincount(key, minlength=nt * nt * nw)))
        ctx.particles_advance(ptk.AB2, 1e-2, 2)
    ctx.close()


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("scheme", ["EULER", "HEUN", "AB2", "AB4"])
def test_many_movers_on_every_route(ptk, monkeypatch, storage, scheme):
    """Steps of about a cell: most particles change bins at each, the history
    with them.  One-shot calls, resident ones, and a field of two times."""
    print(f"[routes] many movers, {storage} {scheme}", flush=True)
    N, n, dt = 26, 30_011, L / 26
    u, u2 = field(N, 4, storage), field(N, 5, storage)
    X0 = positions(N, n, 7)
    sch = getattr(ptk, scheme)
    depth = ptk.AB_ORDER.get(sch, 0)

    def run(route):
        ctx = context(ptk, monkeypatch, route)
        ctx.set_field(u, K.SPLINE, 6, 1, storage=getattr(ptk, storage.upper()))
        v = ctx.vel_dtype()
        res = []
        for resident in (False, True):
            X, g = X0.clone(), torch.zeros((n, 3, 3), dtype=v, device=DEV)
            h = torch.zeros((depth, n, 3), dtype=v, device=DEV) if depth else None
            if resident:
                ctx.particles_load(X, hist_depth=depth)
                ctx.particles_advance(sch, dt, 5, grad_out=g)
                assert ctx.particles_store(X, hist=h) == depth
            else:
                assert ctx.advance(X, sch, dt, 5, hist=h, grad_out=g) == depth
            res += [X, g] + ([h] if depth else [])
        g = torch.zeros((n, 3, 3), dtype=v, device=DEV)
        X = torch.empty_like(X0)
        for f in (u2, u, u2):
            ctx.set_field_next(f)
            ctx.particles_step_next_field(dt, grad_out=g)
            ctx.particles_store(X, hist=h)
            res += [X.clone(), g.clone()]
        ctx.close()
        return res

    ref = run("direct")
    for route in ("sorted", "sweep"):
        for i, (a, b) in enumerate(zip(run(route), ref)):
            assert torch.equal(a, b), (route, i)


@pytest.mark.parametrize("route", ROUTES)
def test_scratch_of_a_call(ptk, monkeypatch, route):
    """A call needs its four arrays of keys and values, the histogram and the
    offsets, however its particles are evaluated: it fits a device-memory cap
    that leaves room for no fifth array of 4 bytes a particle."""
    N, n = 16, 100_003
    print(f"[routes] scratch, {route}", flush=True)
    grown = lambda b: (b + b // 8 + 255) // 256 * 256
    row = ((N + 3) * 12 + 48 + 63) // 64 * 64
    cap = grown(row * (N + 3) ** 2 + 64) + 4 * grown(4 * n) + grown(4 * 256 * -(-n // 2048)) + (64 << 10)
    monkeypatch.setenv("PTK_TEST_MAX_BYTES", str(cap))
    ctx = context(ptk, monkeypatch, route)
    monkeypatch.delenv("PTK_TEST_MAX_BYTES")
    ctx.set_field(field(N, 1, "f32"), ptk.LAGRANGE, 4, 0, storage=ptk.F32)
    X = positions(N, n, 3)
    ctx.interpolate(X)
    ctx.interpolate_gradient(X)
    keys = geometry.bin_keys(X.cpu().numpy(), N, 12, 5)
    for _ in range(2):
        assert np.array_equal(ctx.binning()[0].cpu().numpy(), geometry.stable_order(keys))
    ctx.close()


@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("N", [16, 60])
def test_captured_binning_query(ptk, monkeypatch, route, N):
    """ptk_get_binning recorded in a graph (one and two digit passes): every
    replay gives the binning of the last call, as the eager query between them."""
    n = 5003
    print(f"[routes] captured binning query, {route} N={N}", flush=True)
    ctx = context(ptk, monkeypatch, route)
    ctx.set_field(field(N, 1, "f32"), ptk.LAGRANGE, 4, 0, storage=ptk.F32)
    X = positions(N, n, 1)
    ctx.interpolate(X)
    perm = torch.zeros(n, dtype=torch.int32, device=DEV)
    off = torch.zeros(geometry.n_bins(N, 12, 5) + 1, dtype=torch.int32, device=DEV)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        assert ptk.lib.ptk_get_binning(ctx._h, perm.data_ptr(), off.data_ptr(), side.cuda_stream) == ptk.OK
    for rep in range(4):
        if rep == 2:
            X = positions(N, n, 2)
            ctx.interpolate(X)
        order = geometry.stable_order(geometry.bin_keys(X.cpu().numpy(), N, 12, 5))
        perm.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(perm.cpu().numpy(), order), rep
        eager, eoff, _, _ = ctx.binning()
        assert np.array_equal(eager.cpu().numpy(), order), rep
        assert torch.equal(off, eoff)
    ctx.close()


@pytest.mark.parametrize("kind", ["tracers", "axes", "inertia"])
@pytest.mark.parametrize("scheme", ["HEUN", "AB3"])
def test_steps_through_every_route_in_turn(ptk, kind, scheme):
    """A resident state whose field's kernel and storage change: swept, direct
    and in bin order by the rule, in runs shorter and longer than a sort lasts,
    agrees with the rows of a set that is always read directly."""
    print(f"[routes] in turn: {kind} {scheme}", flush=True)
    N, n, k = 64, 300_000, 500
    u = field(N, 8, "f32")
    g = torch.Generator(device=DEV).manual_seed(5)
    X0 = (torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64) * 3 - 1) * L
    p0 = torch.nn.functional.normalize(torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64))
    sch = getattr(ptk, scheme)
    depth = ptk.AB_ORDER.get(sch, 0)

    def run(X, p):
        ctx = ptk.Context(0)
        m = X.shape[0]
        h = torch.zeros((depth, m, 3), device=DEV) if depth else None
        ph, vh = (torch.zeros((depth, m, 3), device=DEV, dtype=torch.float64) for _ in range(2))
        for e, (fam, I, s, storage) in enumerate([(K.SPLINE, 8, 2, ptk.F32), (K.LAGRANGE, 4, 0, ptk.F32),
                                                  (K.SPLINE, 6, 1, ptk.F32), (K.SPLINE, 8, 2, ptk.BF16),
                                                  (K.LAGRANGE, 4, 0, ptk.F32), (K.SPLINE, 8, 2, ptk.F32)]):
            ctx.set_field(u, fam, I, s, storage=storage)
            if e == 0:
                ctx.particles_load(X, hist_depth=depth)
                if kind == "axes":
                    ctx.particles_set_orientation(p, 0.7)
                elif kind == "inertia":
                    ctx.particles_set_inertia(p, 0.2)
            for c in (3, 7, 12):
                ctx.particles_advance(sch, 2e-3, c)
        ctx.particles_store(X, hist=h)
        if kind == "axes":
            ctx.particles_get_orientation(p, hist=ph)
        elif kind == "inertia":
            ctx.particles_get_inertia(p, v_hist=vh, r_hist=ph)
        ctx.close()
        return [X, p] + [t.transpose(0, 1) for t in (ph, vh)] + ([h.transpose(0, 1)] if depth else [])

    a, b = run(X0.clone(), p0.clone()), run(X0[:k].clone(), p0[:k].clone())
    for x, y in zip(a, b):
        assert torch.equal(x[:k], y)
