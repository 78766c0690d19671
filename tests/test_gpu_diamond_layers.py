"""The diamond space on more layers than one launch of 64 x 32 tiles holds
(4194305 of 65 x 33 cells, two such tiles to a diagonal): 64 x 64 tiles serve
them, every layer as a single one."""
import pytest

import paper_1207_1746_amd as G

pytestmark = pytest.mark.gpu


def test_diamond_more_layers_than_a_launch_of_small_tiles(ctx):
    import torch
    nl, ny, nx = 2 ** 22 + 1, 33, 65
    one = torch.randn((1, ny, nx), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    u1 = ctx.grid((1, ny, nx), G.F32, halo=1, ndim=2, data=one)
    ctx.do_diamond(G.K_GS2D, [u1], [u1], p=(1.3, 0.01))
    u = ctx.grid((nl, ny, nx), G.F32, halo=1, ndim=2)
    u.view.copy_(one.expand(nl, ny, nx))
    ctx.do_diamond(G.K_GS2D, [u], [u], p=(1.3, 0.01))
    step = 1 << 18
    assert all(bool((u.view[z:z + step] == u1.view[0]).all()) for z in range(0, nl, step))
    del u
    torch.cuda.empty_cache()
