"""The tuner against a stub context and timer: the library's own choice is timed
with no tile installed, stays unless a candidate clearly beats it, and is what
the cache brings back; blocked kinds are recorded by their levels; records of
kinds whose tiles changed their meaning are not taken up."""
import types

import pytest

import paper_1207_1746_amd as G
from paper_1207_1746_amd import autotune as AT

DEFAULT = (1, 16, 7)


class _Ctx:
    """Tiles by kind; do_all records the tile a call runs with."""
    stream = None

    def __init__(self):
        self.tiles, self.ran = {}, None

    def tile_get(self, kind, g):
        return self.tiles.get(kind, DEFAULT)

    def tile_set(self, kind, g, tile):
        self.tiles[kind] = tuple(tile)

    def tile_unset(self, kind, g):
        self.tiles.pop(kind, None)

    def do_all(self, kind, ins, outs, p=(), terms=None):
        self.ran = self.tiles.get(kind)
        if self.ran == (9, 9, 9):
            raise G.GsclError(G.ERR_UNSUPPORTED, "stub")


def _grid():
    return types.SimpleNamespace(desc=G.make_desc((20, 30, 40), G.F64))


def _tuner(monkeypatch, tmp_path, ms):
    ctx = _Ctx()

    def time_call(fn, reps=10, warmup=2, stream=None):
        fn()
        return ms(ctx.ran)

    monkeypatch.setattr(AT, "time_call", time_call)
    return AT.Tuner(ctx, str(tmp_path / "tiles.json")), ctx


@pytest.mark.parametrize("kind,p", [(G.K_IMG_BOX5_LAP, (4,)), (G.K_WJACOBI_TB, (0.8, 0.1, 4)), (G.K_WJACOBI, (0.8, 0.1))])
@pytest.mark.parametrize("best,own", [(0.5, False), (0.96, False), (0.98, True), (1.5, True)])
def test_own_choice_is_timed_and_kept(monkeypatch, tmp_path, kind, p, best, own):
    t, ctx = _tuner(monkeypatch, tmp_path, lambda tile: 1.0 if tile is None else best if tile[2] == 8 else 2.0)
    ctx.tile_set(kind, _grid(), (1, 16, 3))  # left by an earlier tuning
    rec = t.tune(kind, [_grid()], [_grid()], p=p)
    assert rec["own"] is own and rec["own_us"] == 1000.0
    assert (ctx.tiles.get(kind) is None) is own
    assert tuple(rec["tile"]) == ctx.tile_get(kind, _grid())
    assert len(rec["tried"]) == len(AT.candidates(kind, G.F64, 20))
    t.save()
    t2 = AT.Tuner(ctx, str(tmp_path / "tiles.json"))
    for again in (lambda: t2.apply(kind, _grid()), lambda: t2.tune(kind, [_grid()], [_grid()], p=p)):
        ctx.tile_set(kind, _grid(), (1, 16, 3))
        assert again()
        assert ctx.tile_get(kind, _grid()) == tuple(rec["tile"]) and (ctx.tiles.get(kind) is None) is own


@pytest.mark.parametrize("kind,head", [(G.K_WJACOBI_TB, (0.8, 0.1)), (G.K_RBGS_TB, (0.8, 0.1, 0))])
def test_blocked_records_by_levels(monkeypatch, tmp_path, kind, head):
    t, ctx = _tuner(monkeypatch, tmp_path, lambda tile: 1.0 if tile is None else 0.5 if tile[2] == 8 else 2.0)
    t.tune(kind, [_grid()], [_grid()], p=head + (2,))
    ctx.tiles.clear()
    assert not t.apply(kind, _grid(), p=head + (4,)) and not ctx.tiles
    assert t.apply(kind, _grid(), p=head + (2,)) and ctx.tiles[kind][2] == 8
    assert t.apply(kind, _grid())


def test_candidates_hold_the_library_image_chunks():
    assert {1, 2, 4} <= {cy for _, _, cy in AT.candidates(G.K_IMG_BOX5_LAP, G.U8, 1)}


def test_earlier_records(monkeypatch, tmp_path):
    t, ctx = _tuner(monkeypatch, tmp_path, lambda tile: 1.0)
    for kind in (G.K_WJACOBI_TB, G.K_IMG_BOX5_LAP, G.K_WJACOBI):
        t.table[f"{t.arch}|{kind}|{G.F64}|40x30x20"] = {"tile": [1, 16, 5], "us": 1.0, "tried": []}
    assert not t.apply(G.K_WJACOBI_TB, _grid()) and not t.apply(G.K_IMG_BOX5_LAP, _grid())
    assert t.apply(G.K_WJACOBI, _grid()) and ctx.tiles == {G.K_WJACOBI: (1, 16, 5)}


def test_no_candidate_runs(monkeypatch, tmp_path):
    t, ctx = _tuner(monkeypatch, tmp_path, lambda tile: 1.0)
    with pytest.raises(RuntimeError):
        t.tune(G.K_WJACOBI, [_grid()], [_grid()], p=(0.8, 0.1), cands=[(9, 9, 9)])
    assert not ctx.tiles
