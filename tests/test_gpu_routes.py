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
