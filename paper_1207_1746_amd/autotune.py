"""Tile autotuner for the tiled do_all kernels (autotuning is the paper's
stated future work, Section 2 and Section 6).

For one operator kind and one set of grid extents it times the library's own
choice and every candidate tile shape (V elements per lane, NW waves per block,
cz planes per block) with HIP events.  A candidate that beats the library's
choice by more than the timings' spread is installed in the context with
``gscl_tile_set``; otherwise the choice stays with the library, which for the
blocked kinds balances each launch and for small images takes another kernel.
The outcome is recorded in a JSON cache keyed by (gfx arch, kind, dtype,
extents; the blocked kinds also by their levels).  Outputs do not depend on the
tile shape (only the fused-reduction rounding order does), so tuning never
changes a do_all result.

For the batched executor it picks, per request-size bucket, the z chunks of
the one-sweep and blocked-pass tiles (``gscl_batch_tile_rule``) by timing
steps of a batch filled with requests of the bucket's size, and caches the
rule under (gfx arch, precision, method, step and pass lengths, bucket).
"""
from __future__ import annotations

import itertools
import json
import os
from typing import Callable, Iterable, Sequence

import paper_1207_1746_amd as G

DEFAULT_CACHE = os.environ.get("GSCL_TILE_CACHE",
                               os.path.join(os.path.expanduser("~"), ".cache", "gscl", "tiles.json"))

RADIUS2 = (G.K_VC13_APPLY, G.K_VC13_JACOBI, G.K_VC13_RESID)


BLOCKED = (G.K_WJACOBI_TB, G.K_RBGS_TB)

# request-size buckets of the batched executor: (largest extent, cube side
# timed for the bucket)
BATCH_BUCKETS = ((48, 40), (96, 80), (144, 128), (192, 176))


def candidates(kind: int, dtype: int, nz: int) -> list[tuple[int, int, int]]:
    """Tile shapes that have an instantiated kernel for this kind and dtype."""
    if kind == G.K_IMG_BOX5_LAP:
        return [(4, 4, cy) for cy in (1, 2, 4, 8, 16, 32, 64)]
    if kind in BLOCKED:
        # fixed block shape: only the z chunk (output planes) varies
        return [(1, 16, cz) for cz in (1, 2, 3, 4, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64) if cz <= max(nz, 1)]
    if kind in RADIUS2:
        # one-field operators run NW = 4 only; shapes without a kernel are
        # skipped by the tuner (the launch reports them as unsupported)
        vs, nws = ((1,) if dtype == G.F64 else (1, 2)), (4, 6, 8)
    elif dtype == G.F64:
        vs, nws = (1, 2), (4, 8)
    else:
        vs, nws = (1, 2, 4), (4, 8)
    czs = [c for c in (1, 2, 4, 8, 16, 32, 64) if c <= max(nz, 1)]
    return [(v, nw, cz) for v, nw, cz in itertools.product(vs, nws, czs)]


def _key(arch: str, kind: int, g: "G.Grid", p: Sequence[float] = ()) -> str:
    d = g.desc
    key = f"{arch}|{kind}|{d.dtype}|{d.n[0]}x{d.n[1]}x{d.n[2]}"
    if kind in BLOCKED:  # the levels of a pass: the last parameter; 4 where it is not known
        at = 2 if kind == G.K_WJACOBI_TB else 3
        key += f"|k{int(p[at]) if len(p) > at else 4}"
    # (kinds whose tiles mean something else than in earlier records)
    return key + "|r2" if kind in BLOCKED or kind == G.K_IMG_BOX5_LAP else key


def _arch() -> str:
    import torch
    try:
        return torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    except Exception:
        return "gfx950"


def time_call(fn: Callable[[], None], reps: int = 10, warmup: int = 2, stream=None) -> float:
    """Mean milliseconds of fn() with HIP events on `stream` (the stream fn
    launches on; default the current stream)."""
    import torch
    for _ in range(warmup):
        fn()
    s = torch.cuda.Event(enable_timing=True)
    e = torch.cuda.Event(enable_timing=True)
    s.record(stream)
    for _ in range(reps):
        fn()
    e.record(stream)
    e.synchronize()
    return s.elapsed_time(e) / reps


class Tuner:
    def __init__(self, ctx: "G.Context", cache_path: str | None = DEFAULT_CACHE):
        self.ctx = ctx
        self.cache_path = cache_path
        self.arch = _arch()
        self.table: dict[str, dict] = {}
        if cache_path and os.path.exists(cache_path):
            with open(cache_path) as f:
                self.table = json.load(f)

    def tune(self, kind: int, ins: Sequence["G.Grid"], outs: Sequence["G.Grid"], p: Iterable[float] = (),
             terms=None, cands: list | None = None, reps: int = 10, force: bool = False) -> dict:
        """Pick the fastest tile for do_all(kind, ins, outs, p) and install it
        (none where the library's own choice is as fast: record "own").  A chunk
        installed for a blocked kind holds for every number of levels."""
        ref = ins[0]
        p = tuple(p)
        key = _key(self.arch, kind, ref, p)
        if not force and key in self.table:
            self._install(kind, ref, self.table[key])
            return self.table[key]
        cands = cands or candidates(kind, ref.desc.dtype, ref.desc.n[2])

        def time_it():
            try:
                return time_call(lambda: self.ctx.do_all(kind, ins, outs, p=p, terms=terms), reps=reps,
                                 stream=self.ctx.stream)
            except G.GsclError:  # no kernel for the shape
                return None

        self.ctx.tile_unset(kind, ref)
        own_tile, own = self.ctx.tile_get(kind, ref), time_it()
        results = []
        for tile in cands:
            self.ctx.tile_set(kind, ref, tile)
            ms = time_it()
            if ms is not None:
                results.append((ms, tile))
        if own is None or not results:
            self.ctx.tile_unset(kind, ref)
            raise RuntimeError("no tile candidate ran")
        results.sort()
        ms, tile = results[0]
        # the same call timed twice differs by up to some percent
        keep = ms > 0.97 * own
        rec = {"tile": list(own_tile if keep else tile), "us": (own if keep else ms) * 1e3, "own": keep,
               "own_us": round(own * 1e3, 2), "tried": [[list(t), round(m * 1e3, 2)] for m, t in results]}
        self._install(kind, ref, rec)
        self.table[key] = rec
        return rec

    def _install(self, kind: int, grid: "G.Grid", rec: dict):
        if rec.get("own"):
            self.ctx.tile_unset(kind, grid)
        else:
            self.ctx.tile_set(kind, grid, tuple(rec["tile"]))

    def apply(self, kind: int, grid: "G.Grid", p: Sequence[float] = ()) -> bool:
        """Install the cached outcome for (kind, grid extents; blocked kinds: the
        levels in p, else 4 or the most there is a record for) if there is one."""
        keys = [_key(self.arch, kind, grid, p)]
        if kind in BLOCKED and not len(p):
            keys = [_key(self.arch, kind, grid, (0, 0, k) if kind == G.K_WJACOBI_TB else (0, 0, 0, k))
                    for k in (4, 3, 2, 1)]
        for key in keys:
            if key in self.table:
                self._install(kind, grid, self.table[key])
                return True
        return False

    def tune_batch(self, precision: int = G.PREC_F32_IR, method: int = G.BATCH_JACOBI,
                   sweeps_per_step: int = 64, sweeps_per_pass: int = 4, buckets=BATCH_BUCKETS,
                   slots: int = 8, reps: int = 3, force: bool = False) -> list[tuple]:
        """Tile rule [(edge, cz, tb_cz), ...] for a batch of this
        configuration: per bucket, the (cz, tb_cz) whose step is fastest on a
        batch of `slots` requests of the bucket's size (never converging
        during the timing)."""
        import numpy as np
        import torch
        ctx = self.ctx
        rules = []
        for edge, n in buckets:
            key = f"batch|{self.arch}|p{precision}|m{method}|S{sweeps_per_step}|k{sweeps_per_pass}|{edge}"
            if not force and key in self.table:
                rules.append((edge, *self.table[key]["rule"]))
                continue
            shape = (n, n, n)
            f = ctx.grid(shape, G.F64, halo=0, data=np.random.default_rng(n).standard_normal(shape))
            us = [ctx.grid(shape, G.F64, halo=1) for _ in range(slots)]
            czs = (4, 8, 16)
            tbs = (4, 8, 16, 32) if sweeps_per_pass > 1 else (0,)
            results = []
            for cz in czs:
                for tb in tbs:
                    probe = G.Batch(ctx, max_slots=slots, precision=precision, hbm_budget=1 << 20, method=method,
                                    sweeps_per_step=sweeps_per_step, sweeps_per_pass=sweeps_per_pass)
                    budget = int(slots * probe.footprint(shape) * 1.25) + (64 << 20)
                    probe.close()
                    b = G.Batch(ctx, max_slots=slots, precision=precision, sweeps_per_step=sweeps_per_step,
                                rtol=1e-300, hbm_budget=budget, method=method, omega=6 / 7 if method == G.BATCH_JACOBI
                                else 0.0, sweeps_per_pass=sweeps_per_pass, max_sweeps=10 ** 9)
                    b.set_tile_rule([(edge, cz, tb)])
                    for u in us:
                        u.fill(0.0)
                        assert b.admit(u, f, 1.0 / (n + 1) ** 2) is not None
                    ms = time_call(b.step, reps=reps, warmup=1, stream=ctx.stream)
                    b.close()
                    results.append((ms, (cz, tb)))
            del us, f
            torch.cuda.empty_cache()
            results.sort()
            ms, best = results[0]
            self.table[key] = {"rule": list(best), "ms_per_step": round(ms, 4),
                               "tried": [[list(t), round(m, 4)] for m, t in results]}
            rules.append((edge, *best))
        return rules

    def save(self, path: str | None = None):
        path = path or self.cache_path
        if not path:
            return
        os.makedirs(os.path.dirname(os.path.abspath(path)), exist_ok=True)
        tmp = path + ".tmp"
        with open(tmp, "w") as f:
            json.dump(self.table, f, indent=1, sort_keys=True)
        os.replace(tmp, path)
