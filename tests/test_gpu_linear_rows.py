"""GPU parity of the LINEAR do_all at the edges of its row and vector split
(one or two rows per wave, 1, 2 or 4 points per lane): every boundary rule,
each grid with its own, offsets up to the declared halo, several outputs, a
coefficient grid, and an output that is an input read at the core element.

Tolerance: each point is a sum of n fused multiply-adds of products of two
values and a weight, so |g - o| <= 2 n eps sum |w| max|in|^2 (eps the
rounding unit of the grid type; the oracle's own FP64 error is below it for
FP32 and of the same size for FP64)."""
import numpy as np
import pytest

import oracle
import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu

# (1, 2 and 4 points per lane) x (one and two rows per wave), at and around
# whole vectors, waves and row groups
SHAPES = [(2, 3, 1), (5, 9, 63), (3, 7, 64), (4, 11, 65), (3, 5, 129), (2, 9, 257), (130, 131, 66), (129, 130, 130),
          (67, 127, 261)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dt", [G.F64, G.F32])
@pytest.mark.parametrize("ndim", [3, 2])
def test_linear_rows_match_oracle(ctx, shape, dt, ndim):
    g = np.random.default_rng(sum(shape) + 10 * dt + ndim)
    np_t = np.float64 if dt == G.F64 else np.float32
    arrs = [g.standard_normal(shape).astype(np_t) for _ in range(3)]
    bcs = [G.DIRICHLET, G.PERIODIC, G.CLAMP]
    bcv = [0.75, 0.0, 0.0]
    offs = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (2, -1, 0), (-3, 0, 1), (0, 1, 0), (0, -2, -1), (4, 4, -4), (-4, 1, 2)]
    terms = []
    for k, (dx, dy, dz) in enumerate(offs):
        for gi in range(3):
            # the third grid is also a coefficient; weights exact in FP32
            terms.append((k % 2, gi, dx, dy, dz if ndim == 3 else 0, (k - 3.5) / 8, 2 if (k + gi) % 3 == 0 else -1))
    ins = [ctx.grid(shape, dt, halo=4, bc=bcs[i], bc_value=bcv[i], ndim=ndim, data=a) for i, a in enumerate(arrs)]
    outs = [ctx.grid(shape, dt, halo=0, ndim=ndim) for _ in range(2)]
    r = ctx.do_all(G.K_LINEAR, ins, outs, terms=terms, reduce=(G.R_MAXABS, G.RV_UPDATE))
    exp = oracle.linear(ndim, [a.astype(np.float64) for a in arrs], terms, 2, bcs, bcv)
    top = max(np.abs(a).max() for a in arrs)
    eps = 2.0 ** -53 if dt == G.F64 else 2.0 ** -24
    tol = 2 * len(terms) * eps * sum(abs(t[5]) for t in terms) * max(top, 1.0) ** 2
    for o, e in zip(outs, exp):
        assert np.abs(o.numpy().astype(np.float64) - e.reshape(shape)).max() <= tol
    got0 = outs[0].numpy().astype(np.float64)
    assert r == np.abs(got0 - arrs[0].astype(np.float64)).max()


def test_linear_output_may_be_a_pointwise_input(ctx):
    # out[0] is in[1], read at the core element only: the second output's term
    # sees the value the first output's store left there (one thread per point)
    shape = (40, 66, 131)
    g = np.random.default_rng(9)
    a, b = g.standard_normal(shape), g.standard_normal(shape)
    ga, gb = ctx.grid(shape, G.F64, halo=1, data=a), ctx.grid(shape, G.F64, halo=0, data=b)
    go = ctx.grid(shape, G.F64, halo=0)
    terms = [(0, 0, 1, 0, 0, 1.0, -1), (0, 1, 0, 0, 0, 2.0, -1), (1, 1, 0, 0, 0, 4.0, -1)]
    ctx.do_all(G.K_LINEAR, [ga, gb], [gb, go], terms=terms)
    first = np.zeros(shape)
    first[:, :, :-1] = a[:, :, 1:]
    first += 2.0 * b
    assert np.array_equal(gb.numpy(), first)
    assert np.array_equal(go.numpy(), 4.0 * first)
