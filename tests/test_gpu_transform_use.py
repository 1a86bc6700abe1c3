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


@pytest.mark.parametrize("storage", ["F64", "F32", "BF16", "F16"])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("N", [64, 128])
def test_device_memory_of_a_transform(ptk, monkeypatch, N, prec, storage):
    """Beside the field, the transform takes its own buffer alone (rows of the
    half spectrum on whole 128-byte lines) and small tables: it fits a cap that
    leaves room for no grid of real values."""
    print(f"[spectrum] memory, N={N} {prec} -> {storage}", flush=True)
    grown = lambda b: (b + b // 8 + 255) // 256 * 256
    cb = 16 if prec == "f64" else 8
    node = {"F64": 24, "F32": 12}.get(storage, 6)
    row = ((N + 7) * node + 48 + 63) // 64 * 64
    cap = grown(N * N * (-(-3 * (N // 2 + 1) * cb // 128) * 128)) + grown(row * (N + 7) ** 2 + 64) + (256 << 10)
    spec = spectrum(N, prec)
    ref = ptk.Context(0)
    ref.set_field_spectral(spec, ptk.SPLINE, 8, 2, storage=getattr(ptk, storage))
    monkeypatch.setenv("PTK_TEST_MAX_BYTES", str(cap))
    ctx = ptk.Context(0)
    monkeypatch.delenv("PTK_TEST_MAX_BYTES")
    ctx.set_field_spectral(spec, ptk.SPLINE, 8, 2, storage=getattr(ptk, storage))
    assert torch.equal(ctx.get_field(), ref.get_field()) and ctx.field_scale() == ref.field_scale()
    ctx.close()
    ref.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_transforms_recorded_in_graphs_and_eager_ones_in_turn(ptk, prec):
    """A transform recorded in a graph before any was run at its size, eager ones
    of that size and another before and between its replays: every field is
    the one an eager call on a context of its own gives."""
    print(f"[spectrum] recorded, {prec}", flush=True)
    spec = {N: spectrum(N, prec, N) for N in (64, 128)}
    ref = {}
    for N in spec:
        ctx = ptk.Context(0)
        ctx.set_field_spectral(spec[N], ptk.SPLINE, 8, 2, storage=ptk.F64, kind=ptk.SPEC_VORTICITY)
        ref[N] = ctx.get_field()
        ctx.close()
    ctx = ptk.Context(0)

    def eager(N):
        ctx.set_field_spectral(spec[N], ptk.SPLINE, 8, 2, storage=ptk.F64, kind=ptk.SPEC_VORTICITY)
        torch.cuda.synchronize()
        assert torch.equal(ctx.get_field(), ref[N])

    eager(128)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        ctx.set_field_spectral(spec[64], ptk.SPLINE, 8, 2, storage=ptk.F64, kind=ptk.SPEC_VORTICITY)
    eager(64)
    for other in (64, 128, 128, 64):
        eager(other)
        eager(64)  # (the context's own idea of its field is of the recorded size again)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ctx.get_field(), ref[64])
    ctx.close()
