"""Batches around and above 64 slots, the number the kernels look a tile's slot
up in at a time: every request's answer is bit for bit the one it has alone,
while slots finish, stay finished for a while and are reused."""
import numpy as np
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu

SHAPES = [(3, 4, 5), (9, 2, 7), (1, 1, 1), (12, 13, 14), (5, 26, 60), (17, 3, 2), (8, 8, 8)]


def _serve(ctx, which, max_slots, **kw):
    """Shapes SHAPES[i] for i in which, in arrival order: [(u, sweeps)]."""
    b = G.Batch(ctx, max_slots=max_slots, sweeps_per_step=8, rtol=1e-6, hbm_budget=1 << 30, **kw)
    f = {i: ctx.grid(SHAPES[i], G.F64, halo=0, data=np.random.default_rng(i).standard_normal(SHAPES[i]))
         for i in set(which)}
    us = [ctx.grid(SHAPES[i], G.F64, halo=1).fill(0.0) for i in which]
    slots, out, queue, polls = {}, [None] * len(which), list(range(len(which))), 0
    while slots or queue:
        while queue and (s := b.admit(us[queue[0]], f[which[queue[0]]], 0.01)) is not None:
            slots[s] = queue.pop(0)
        b.step()
        polls += 1
        done = b.poll()
        if polls % 3 and len(done) < len(slots):
            continue  # finished slots stay in the table for a while
        for s in done:
            k = slots.pop(s)
            st = b.retire(s)
            assert st["state"] == 2
            out[k] = (us[k].numpy(), st["sweeps"])
        assert polls < 10000
    b.close()
    return out


@pytest.mark.parametrize("kw", [dict(precision=G.PREC_F64), dict(precision=G.PREC_F64, sweeps_per_pass=4),
                                dict(precision=G.PREC_F32_IR, sweeps_per_pass=4),
                                dict(precision=G.PREC_F64, method=G.BATCH_RBGS, omega=0.0, sweeps_per_pass=2)])
def test_many_slots_equal_alone(ctx, kw):
    alone = [_serve(ctx, [i], 1, **kw)[0] for i in range(len(SHAPES))]
    for count, slots in ((64, 64), (65, 65), (300, 130)):
        which = [(3 * k + k // 5) % len(SHAPES) for k in range(count)]
        for k, (u, sweeps) in enumerate(_serve(ctx, which, slots, **kw)):
            assert sweeps == alone[which[k]][1], (count, k)
            assert np.array_equal(u, alone[which[k]][0]), (count, k)


def test_largest_table(ctx):
    with pytest.raises(G.GsclError) as e:
        G.Batch(ctx, max_slots=4097)
    assert e.value.code == G.ERR_ARG
    alone = _serve(ctx, [0], 1, sweeps_per_pass=4)[0]
    for u, sweeps in _serve(ctx, [0] * 4096, 4096, sweeps_per_pass=4):
        assert sweeps == alone[1] and np.array_equal(u, alone[0])
