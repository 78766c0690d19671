"""Fused reductions of the blocked kinds through gscl_do_all_noalloc: the same
launch as gscl_do_all, so outputs and reduced values agree bit for bit; also
where the launch has more blocks than GSCL_NOALLOC_PARTIALS while its count
(tiles of exactly k ghost columns) is at the limit."""
import numpy as np
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu

REDUCE = ((G.R_L2, G.RV_UPDATE), (G.R_SUMSQ, G.RV_RESIDUAL))


def _args(kind, k):
    return (0.8, 0.1, k) if kind == G.K_WJACOBI_TB else (1.6, 0.1, 1, k)


@pytest.mark.parametrize("dt", [G.F64, G.F32])
@pytest.mark.parametrize("kind", [G.K_WJACOBI_TB, G.K_RBGS_TB])
def test_blocked_noalloc_matches_do_all(ctx, kind, dt):
    rng = np.random.default_rng(5)
    shape = (37, 45, 119)
    u, f = (ctx.grid(shape, dt, halo=1, data=rng.standard_normal(shape)) for _ in range(2))
    a, b = ctx.grid(shape, dt, halo=1), ctx.grid(shape, dt, halo=1)
    for cz in (0, 5):
        if cz:
            ctx.tile_set(kind, u, (1, 16, cz))
        for k in (1, 2, 3, 4):
            for red in REDUCE:
                ra = ctx.do_all(kind, [u, f], [a], p=_args(kind, k), reduce=red)
                rb = ctx.do_all(kind, [u, f], [b], p=_args(kind, k), reduce=red, noalloc=True)
                assert ra == rb and ra > 0, (k, red, cz)
                assert np.array_equal(a.numpy(), b.numpy()), (k, red, cz)
    ctx.tile_clear()


@pytest.mark.parametrize("kind", [G.K_WJACOBI_TB, G.K_RBGS_TB])
def test_blocked_noalloc_at_the_limit(ctx, kind):
    """15872 x 7680: 256 x 256 tiles of 62 x 30 points, 265 x 256 of a pair layout's 60 x 30."""
    import torch
    shape = (1, 7680, 15872)
    u = ctx.grid(shape, G.F32, halo=1)
    u.storage.copy_(torch.rand(u.storage.shape, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda"))
    a, b = ctx.grid(shape, G.F32, halo=1), ctx.grid(shape, G.F32, halo=1)
    ra = ctx.do_all(kind, [u], [a], p=_args(kind, 1), reduce=REDUCE[0])
    rb = ctx.do_all(kind, [u], [b], p=_args(kind, 1), reduce=REDUCE[0], noalloc=True)
    assert ra == rb and ra > 0
    assert torch.equal(a.view, b.view)
    wide = ctx.grid((1, 7680, 15873), G.F32, halo=1).fill(0.0)
    out = ctx.grid((1, 7680, 15873), G.F32, halo=1)
    with pytest.raises(G.GsclError) as e:
        ctx.do_all(kind, [wide], [out], p=_args(kind, 1), reduce=REDUCE[0], noalloc=True)
    assert e.value.code == G.ERR_NOMEM
