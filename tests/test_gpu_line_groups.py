"""Line kernels at the lengths where their groups of cells end (16 requested
ahead on few lines, 8 on many, chunks of 32 along x), in both directions,
against the oracle: the same operations in the same order, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("direction", [1, -1])
@pytest.mark.parametrize("few", [True, False])
def test_line_group_ends(ctx, axis, direction, few):
    rng = np.random.default_rng(axis)
    for n in (1, 15, 16, 17, 31, 32, 33, 49) if few else (1, 7, 8, 9, 33):
        shape = [5, 5, 5] if few else [257, 257, 257]
        shape[2 - axis] = n
        lo, up = (rng.uniform(-1, 1, shape) for _ in range(2))
        di, rhs = 2.5 + rng.uniform(0, 1, shape), rng.standard_normal(shape)
        gs = [ctx.grid(tuple(shape), G.F64, halo=0, data=v) for v in (lo, di, up, rhs)]
        cp, dp, x = (ctx.grid(tuple(shape), G.F64, halo=0) for _ in range(3))
        ctx.do_line(G.K_TRIDIAG_FWD, axis, direction, gs, [cp, dp])
        ctx.do_line(G.K_TRIDIAG_BACK, axis, -direction, [cp, dp], [x])
        ecp, edp = oracle.tridiag_fwd(lo, di, up, rhs, axis, direction)
        assert np.array_equal(cp.numpy(), ecp) and np.array_equal(dp.numpy(), edp), n
        assert np.array_equal(x.numpy(), oracle.tridiag_back(ecp, edp, axis, -direction)), n
        ctx.do_line(G.K_LINE_RECUR, axis, direction, [gs[0], gs[3]], [x], p=(0.5,))
        assert np.array_equal(x.numpy(), oracle.line_recur(lo, rhs, axis, direction, seed=0.5)), n
