"""The library's own inverse transform at every grid size it is built for, and
sizes beside them that take the general one: the stored field, read back,
against the oracle within the transform bound 8 log2(N^3) eps A."""
import numpy as np
import pytest
import torch

from oracle import kernels as K
from oracle import spectral as sp
from synthetic import fields

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ptk(lib):
    return lib


def check(got, w, kind, eps, store):
    ref = sp.grid_field(w, kind)
    tol = 8.0 * np.log2(w.shape[0] ** 3) * eps * sp.absolute_sum(w, kind) + store * np.abs(ref)
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) / tol))


@pytest.mark.parametrize("N", [62, 64, 128])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", ["velocity", "vorticity"])
@pytest.mark.parametrize("storage,I", [("f64", 8), ("f32", 4), ("bf16", 6)])
def test_transform_matches_oracle(ptk, N, prec, kind, storage, I):
    print(f"[transform] N={N} {prec} {kind} -> {storage} I={I}", flush=True)
    w = fields.spectrum_modes(N, kc=N / 3.0, seed=N + I, nyquist=True)
    if prec == "f32":
        w = w.astype(np.complex64).astype(np.complex128)
    spec = torch.from_numpy(w.astype(np.complex64) if prec == "f32" else w).to(DEV)
    k = ptk.SPEC_VORTICITY if kind == "vorticity" else ptk.SPEC_VELOCITY
    code = {"f64": ptk.F64, "f32": ptk.F32, "bf16": ptk.BF16}[storage]
    ctx = ptk.Context(0)
    fam, m = (K.LAGRANGE, 0) if I == 4 else (K.SPLINE, 2)
    ctx.set_field_spectral(spec, fam, I, m, storage=code, kind=k)
    got = ctx.get_field(torch.float64).cpu().numpy() * np.array(ctx.field_scale(), dtype=np.float64)
    eps = 2.0 ** -53 if prec == "f64" else 2.0 ** -24
    store = {"f64": 0.0, "f32": 2.0 ** -24, "bf16": 2.0 ** -8 + 2.0 ** -21}[storage]
    check(got, w, sp.VORTICITY if kind == "vorticity" else sp.VELOCITY, eps, store)
    if storage != "bf16":
        # the halo: a particle in every corner cell interpolates nodes across
        # the faces; against a context given the same grid values
        X = torch.cartesian_prod(*[torch.tensor([1e-3, 2 * np.pi - 1e-3], dtype=torch.float64)] * 3).to(DEV)
        other = ptk.Context(0)
        other.set_field(ctx.get_field(torch.float64), fam, I, m, storage=code)
        for f64 in (torch.float64, torch.float32):
            assert torch.equal(ctx.interpolate(X, out_dtype=f64), other.interpolate(X, out_dtype=f64))
        # the next field of a two-field step goes the same way
        ctx.set_field_next_spectral(spec, k)
        ctx.particles_load(X)
        ctx.particles_step_next_field(0.0)
        assert torch.equal(ctx.get_field(torch.float64), other.get_field(torch.float64))
        other.close()
    ctx.close()


@pytest.mark.parametrize("N,prec", [(256, "f64"), (256, "f32"), (512, "f64"), (512, "f32"), (1024, "f64")])
def test_transform_large_sparse(ptk, N, prec):
    """Spectra of 40 modes up to the last wave number below N/2, at 4 099 nodes
    (the first and last of every axis among them) against the series."""
    print(f"[transform] N={N} {prec}, 40 modes", flush=True)
    k2i, k3i, k1, amp = fields.sparse_spectrum(N, 40, N // 2 - 1, seed=N)
    dt = torch.complex128 if prec == "f64" else torch.complex64
    if prec == "f32":
        amp = amp.astype(np.complex64).astype(np.complex128)
    spec = torch.zeros((N, N, N // 2 + 1, 3), dtype=dt, device=DEV)
    spec[torch.from_numpy(k2i), torch.from_numpy(k3i), torch.from_numpy(k1)] = torch.from_numpy(amp).to(DEV).to(dt)
    ctx = ptk.Context(0)
    ctx.set_field_spectral(spec, K.SPLINE, 8, 2, storage=ptk.F32 if N == 1024 else ptk.F64)
    del spec
    rng = np.random.default_rng(N)
    nodes = rng.integers(0, N, (4099, 3))
    nodes[:8] = [[a, b, c] for a in (0, N - 1) for b in (0, N - 1) for c in (0, N - 1)]
    u = ctx.get_field(torch.float32 if N == 1024 else torch.float64)
    j = torch.from_numpy(nodes).to(DEV)
    got = u[j[:, 2], j[:, 1], j[:, 0]].double().cpu().numpy()
    ref = sp.series_sparse(N, k2i, k3i, k1, amp, nodes)
    A = np.sum(np.abs(amp) * np.where((k1 > 0) & (k1 < N // 2), 2.0, 1.0)[:, None], axis=0)
    tol = 8 * np.log2(N ** 3) * (2.0 ** -53 if prec == "f64" else 2.0 ** -24) * A
    tol = tol + (2.0 ** -24 * np.abs(ref) if N == 1024 else 0.0)
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) / tol))
    ctx.close()
