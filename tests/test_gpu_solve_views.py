"""A Poisson solve whose x and b are columns of one array (interleaved rows, so
their address ranges overlap while no element is shared): small grids solve as
with separate arrays, the same sweeps bit for bit."""
import numpy as np
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 11, 13), (33, 20, 16)])
def test_jacobi_solve_on_interleaved_views(ctx, shape):
    import torch
    nz, ny, nx = shape
    pitch = (32, 32 * ny)
    rhs = np.random.default_rng(4).standard_normal(shape)
    both = torch.zeros(pitch[1] * nz + 32, dtype=torch.float64, device="cuda")
    x = G.Grid(ctx, G.make_desc(shape, G.F64, halo=1, pitch=pitch), both).fill(0.0)
    b = G.Grid(ctx, G.make_desc(shape, G.F64, halo=0, pitch=pitch), both[16:]).upload(rhs)
    u, f = ctx.grid(shape, G.F64, halo=1).fill(0.0), ctx.grid(shape, G.F64, halo=0, data=rhs)
    kw = dict(h2=0.01, rtol=1e-6, check_every=8)
    st, ref = ctx.solve(G.K_WJACOBI, [x], [b], **kw), ctx.solve(G.K_WJACOBI, [u], [f], **kw)
    assert st["sweeps"] == ref["sweeps"]
    assert np.array_equal(x.numpy(), u.numpy())
    assert np.array_equal(b.numpy(), rhs)
