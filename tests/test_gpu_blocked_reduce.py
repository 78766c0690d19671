"""Fused reductions of the blocked passes at the edges of their tiles, against
those of the last of k plain passes: the operand has the same value at every
point, so the largest magnitude is the same to the bit, and the norm differs by
the order of at most n additions on either side (2 n rounding units of the sum
of squares, n of the norm)."""
import numpy as np
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 56, 57, 60, 61, 113])
@pytest.mark.parametrize("dt", [G.F64, G.F32])
@pytest.mark.parametrize("rule", ["dirichlet", "periodic", "redblack"])
def test_blocked_reductions_against_plain_sweeps(ctx, nx, dt, rule):
    rng = np.random.default_rng(nx)
    bc = G.PERIODIC if rule == "periodic" else G.DIRICHLET
    plain, blocked = (G.K_RBGS, G.K_RBGS_TB) if rule == "redblack" else (G.K_WJACOBI, G.K_WJACOBI_TB)
    for ny, nz in ((25, 3), (49, 10), (3, 1), (31, 2)):
        shape = (nz, ny, nx)
        u = ctx.grid(shape, dt, halo=1, bc=bc, bc_value=0.0 if rule == "periodic" else 0.25,
                     data=rng.standard_normal(shape))
        f = ctx.grid(shape, dt, halo=0, data=rng.standard_normal(shape))
        a, b, go = (ctx.grid(shape, dt, halo=1, bc=bc, bc_value=u.desc.bc_value) for _ in range(3))
        for k in (1, 2, 3, 4):
            for rhs in ([f], []):
                for red in ((op, v) for op in (G.R_L2, G.R_MAXABS) for v in (G.RV_OUT0, G.RV_UPDATE, G.RV_RESIDUAL)):
                    a.view.copy_(u.view)
                    for q in range(k):
                        last = red if q == k - 1 else None
                        if rule == "redblack":
                            want = ctx.do_all(plain, [a] + rhs, [a], p=(1.6, 0.1, (1 + q) % 2), reduce=last)
                        else:
                            want = ctx.do_all(plain, [a] + rhs, [b], p=(0.8, 0.1), reduce=last)
                            a, b = b, a
                    p = (1.6, 0.1, 1, k) if rule == "redblack" else (0.8, 0.1, k)
                    for cz in (0, 2):
                        if cz:
                            ctx.tile_set(blocked, u, (1, 16, cz))
                        got = ctx.do_all(blocked, [u] + rhs, [go], p=p, reduce=red)
                        ctx.tile_clear()
                        case = (shape, k, len(rhs), red, cz)
                        assert np.array_equal(go.numpy(), a.numpy()), case
                        if red[0] == G.R_MAXABS:
                            assert got == want, case
                        else:
                            assert abs(got - want) <= nx * ny * nz * 2.0 ** -52 * want, case
