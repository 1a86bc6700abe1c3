"""The ways a call's particles are evaluated (straight from the field, the same
in bin order, the binned sweep), where a call's size or shape changes them.
PTK_TEST_ROUTE, read when a context is made, takes the choice from the rule."""
import numpy as np
import pytest
import torch

from oracle import geometry

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
L = geometry.L


@pytest.fixture(scope="module")
def ptk(lib):
    return lib


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
    """Steps evaluated in bin order re-bin after each of them (but a one-shot
    call's last), with the sweep's results bit for bit; a state that was not
    sorted when it was loaded is sorted first."""
    print(f"[routes] bin order kept: {kind} {scheme} one_shot={one_shot}", flush=True)
    N, n, steps = 24, 9001, 7
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
            ctx.particles_advance(sch, 2e-2, 2)
            ctx.particles_advance(sch, 2e-2, steps - 2, grad_out=gr)
            ctx.particles_store(X, hist=h)
            if kind == "axes":
                ctx.particles_get_orientation(p, hist=ph)
            elif kind == "inertia":
                ctx.particles_get_inertia(p, v_hist=vh, r_hist=ph)
        sorts = ctx.timing_read()["sort"][1]
        ctx.close()
        return sorts, [X, p, gr, ph, vh] + ([h] if depth else [])

    sorts, a = run("sorted")
    assert sorts == 1 + steps - (1 if one_shot else 0)
    swept, b = run("sweep")
    assert swept == sorts + (steps if scheme == "HEUN" else 0)  # (the predictor's bins too)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    none, d = run("direct")
    assert none == 0
    for x, y in zip(a, d):
        assert torch.equal(x, y)
