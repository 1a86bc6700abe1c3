"""The field from a half spectrum as callers may use it: buffers aligned only as
their numbers are, grid sizes and precisions in turn."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ptk(lib):
    return lib


def spectrum(N, prec, seed=1):
    """Of a real random field."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    dt = torch.float64 if prec == "f64" else torch.float32
    w = torch.randn((N, N, N, 3), generator=g, device=DEV, dtype=dt)
    return torch.fft.rfftn(w, dim=(1, 0, 2), norm="forward").contiguous()  # [k2][k3][k1][a] of w[x2][x3][x1][a]


@pytest.mark.parametrize("kind", ["SPEC_VELOCITY", "SPEC_VORTICITY"])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("N", [62, 64, 128])
def test_spectrum_aligned_as_a_real_number(ptk, N, prec, kind):
    print(f"[spectrum] one number off its pair's alignment, N={N} {prec} {kind}", flush=True)
    spec, k = spectrum(N, prec), getattr(ptk, kind)
    ctx = ptk.Context(0)
    ctx.set_field_spectral(spec, ptk.SPLINE, 8, 2, storage=ptk.F64, kind=k)
    ref = ctx.get_field()
    real = torch.view_as_real(spec).reshape(-1)
    off = torch.empty(real.numel() + 1, dtype=real.dtype, device=DEV)
    off[1:] = real
    at = ctypes.c_void_p(off.data_ptr() + off.element_size())
    assert at.value % (2 * off.element_size()) != 0
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    code = ptk.F64 if prec == "f64" else ptk.F32
    kernel = ptk.ptk_kernel(ptk.SPLINE, 8, 2)
    for call in (lambda: ptk.lib.ptk_set_field_spectral(ctx._h, at, N, code, k, ptk.F64, ctypes.byref(kernel), stream),
                 lambda: ptk.lib.ptk_set_field_next(ctx._h, at, N, code, k, stream)):
        assert call() == ptk.OK
        assert torch.equal(ctx.get_field(), ref)
    ctx.particles_load(torch.zeros((1, 3), dtype=torch.float64, device=DEV))
    ctx.particles_step_next_field(0.0)
    assert torch.equal(ctx.get_field(), ref)
    ctx.close()
