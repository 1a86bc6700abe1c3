"""The binning at the sizes where its kernels change shape: single tiles, their
edges, one and two digit passes, and more tiles than one round of the scan of a
histogram row (4096 tiles of 2048 particles)."""
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


def drawn(N, n, seed):
    """Particles at cell centres (their cells are certain) and the cells."""
    cells = np.random.default_rng(seed).integers(0, N, (n, 3))
    return torch.from_numpy((cells + 0.5) * (L / N)).to(DEV), cells


def uniform_field(N):
    return torch.tensor([1.0, 0.5, 0.25], device=DEV).expand(N, N, N, 3).contiguous()


@pytest.mark.parametrize("N,n", [(16, 1), (16, 2047), (16, 2049), (24, 70_001), (60, 500_001), (100, 4097 * 2048 + 5)])
def test_permutation_is_the_stable_sort_of_the_bins(ptk, N, n):
    print(f"[sort] N={N} n={n}", flush=True)
    X, cells = drawn(N, n, 3 * N + n)
    ctx = ptk.Context(0)
    ctx.set_field(uniform_field(N), ptk.LAGRANGE, 4, 0, storage=ptk.F32)
    ctx.interpolate(X)
    perm, off, T, W = ctx.binning()
    ctx.close()
    nt, nw = -(-N // T), -(-N // W)
    key = ((cells[:, 1] // T) * nt + cells[:, 0] // T) * nw + cells[:, 2] // W
    np.testing.assert_array_equal(perm.cpu().numpy(), np.argsort(key, kind="stable"))
    np.testing.assert_array_equal(off.cpu().numpy()[1:], np.cumsum(np.bincount(key, minlength=nt * nt * nw)))


@pytest.mark.parametrize("N,n", [(24, 70_001), (100, 4097 * 2048 + 5)])
def test_rebinned_particles_are_all_found(ptk, N, n):
    """Three Euler steps of 0.4 cells in a uniform flow: most bins change, and a
    particle that is lost, doubled or in a wrong bin shows as an error or in the
    positions (4 roundings of numbers below 16, and FP32 weights that sum to 1
    to 8 ulp: 3 steps of 0.4 L / N at 1e-6)."""
    print(f"[rebin] N={N} n={n}", flush=True)
    X, _ = drawn(N, n, n)
    dt, u = 0.4 * L / N, torch.tensor([1.0, 0.5, 0.25], device=DEV, dtype=torch.float64)
    want = X + 3 * dt * u
    ctx = ptk.Context(0)
    ctx.set_field(uniform_field(N), ptk.LAGRANGE, 4, 0, storage=ptk.F32)
    ctx.particles_load(X)
    ctx.particles_advance(ptk.EULER, dt, 3)
    ctx.particles_store(X)
    ctx.close()
    assert float((X - want).abs().max()) <= 3 * dt * 1e-6 + 2e-14
