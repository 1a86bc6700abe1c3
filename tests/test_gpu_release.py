"""What a context allocates is given back when it is destroyed."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", ["tracers", "axes", "inertia"])
def test_destroyed_contexts_give_their_memory_back(lib, kind):
    """Ten contexts in turn, each with 2 million particles and histories (0.1 GB
    each at least): the free memory after the last is that after the first, to
    64 MB (another process's or the allocator's own granules)."""
    ptk, n = lib, 2_000_000
    print(f"[release] {kind}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(1)
    u = torch.randn((32, 32, 32, 3), generator=g, device=DEV)
    X = torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64)
    V = torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64)
    free = []
    for _ in range(10):
        ctx = ptk.Context(0)
        ctx.set_field(u, ptk.SPLINE, 8, 2, storage=ptk.F32)
        ctx.particles_load(X, hist_depth=4)
        if kind == "axes":
            ctx.particles_set_orientation(V, 0.5)
        elif kind == "inertia":
            ctx.particles_set_inertia(V, 0.5)
        ctx.particles_advance(ptk.AB4, 1e-3, 2)
        ctx.close()
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    assert free[-1] >= free[0] - (64 << 20), free
