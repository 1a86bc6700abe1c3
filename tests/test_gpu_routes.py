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
