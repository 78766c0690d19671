"""Edges of the blocked passes' tiles (64 columns in pairs x 32 rows, ghost
columns in whole pairs): row lengths around a tile's output and odd ones, whose
last pair is half a pair (and, under the periodic rule, split by the wrap),
every number of levels, chunks picked and set, both starts of the red-black
parity.  The reference is k one-level passes of the plain kinds: the same
operator at every point, so the tolerance is zero."""
import numpy as np
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 2, 55, 56, 57, 113])
@pytest.mark.parametrize("dt", [G.F64, G.F32])
@pytest.mark.parametrize("rule", ["dirichlet", "periodic", "redblack"])
def test_blocked_tiles_against_plain_sweeps(ctx, nx, dt, rule):
    rng = np.random.default_rng(nx)
    bc = G.PERIODIC if rule == "periodic" else G.DIRICHLET
    for ny, nz in ((25, 3), (49, 10)):
        shape = (nz, ny, nx)
        u = ctx.grid(shape, dt, halo=1, bc=bc, bc_value=0.0 if rule == "periodic" else 0.25,
                     data=rng.standard_normal(shape))
        f = ctx.grid(shape, dt, halo=0, data=rng.standard_normal(shape))
        go = ctx.grid(shape, dt, halo=1)
        for k in (1, 2, 3, 4):
            for c0 in (0, 1) if rule == "redblack" else (0,):
                a, b = (ctx.grid(shape, dt, halo=1, bc=bc, bc_value=u.desc.bc_value) for _ in range(2))
                a.view.copy_(u.view)
                for q in range(k):
                    if rule == "redblack":
                        ctx.do_all(G.K_RBGS, [a, f], [a], p=(1.6, 0.1, (c0 + q) % 2))
                    else:
                        ctx.do_all(G.K_WJACOBI, [a, f], [b], p=(0.8, 0.1))
                        a, b = b, a
                kind, p = (G.K_RBGS_TB, (1.6, 0.1, c0, k)) if rule == "redblack" else (G.K_WJACOBI_TB, (0.8, 0.1, k))
                for cz in (0, 1, 3):
                    if cz:
                        ctx.tile_set(kind, u, (1, 16, cz))
                    go.fill(-7.0)
                    ctx.do_all(kind, [u, f], [go], p=p)
                    assert np.array_equal(go.numpy(), a.numpy()), (shape, k, c0, cz)
                ctx.tile_clear()
