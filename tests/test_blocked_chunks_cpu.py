"""Host rules of launches, compiled here for the host alone.

A blocked pass: the z chunk it takes, and the count that decides whether its
fused reduction fits the fixed scratch of gscl_do_all_noalloc.  Every admitted
call has at most as many blocks as the scratch holds, around the limit, for
every number of levels and both layouts, with the chunk picked and with one set.

Chunks of grids that share a launch: on a full chip the chunk without a rule or
the rule's, whichever is longer; on few tiles a rule is an upper bound.

The norm of a red-black solve's check: its blocks fit one launch dimension and
the partials of its points, thin grids and the largest among them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHUNKS = r"""
#include <stdio.h>
#include "gscl.h"
#include "tb7.h"
using namespace gk;

int main() {
    const long limit = GSCL_NOALLOC_PARTIALS;
    long admitted = 0, over = 0, bad = 0;
    const int ny[] = {1, 24, 30, 31, 7680, 10950, 16384}, nz[] = {1, 2, 7, 64, 65, 300};
    for (int y : ny)
        for (int z : nz)
            for (int k = 1; k <= TB_KMAX; ++k)
                for (int nominal : {1, 2, 16, 64})
                    for (int set = 0; set < 2; ++set)
                        for (int lay = 0; lay < 4; ++lay) {
                            const bool rb = lay & 1, f64 = lay & 2;
                            // the longest row that is admitted, the one after it, and short ones
                            Geo g{1, y, z, 0, 0, 0, 0.0};
                            const long rest = tb_nominal_blocks(g, k, nominal);
                            const long cols = limit / rest * (64 - 2 * k);
                            for (long x : {1L, 57L, 59L, 61L, cols / 3, cols - 1, cols, cols + 1}) {
                                if (x < 1 || x > 1L << 30) continue;
                                g.nx = (int)x;
                                const bool in = tb_nominal_blocks(g, k, nominal) <= limit;
                                const int cz = tb_launch_chunk(g, k, nominal, set, rb, f64);
                                const long n = tb_blocks(g, k, cz, tb_pairs(f64, rb));
                                if (cz < 1 || (set && cz != nominal)) ++bad;
                                if (!in) continue;
                                ++admitted;
                                over += n > limit;
                                bad += n > 2 * limit;
                            }
                        }
    printf("%ld %ld %ld\n", admitted, over, bad);
    return 0;
}
"""


NORM = r"""
#include <stdio.h>
#include "launch.h"
using namespace gk;

int main() {
    long seen = 0, bad = 0;
    for (long x : {1L, 3L, 127L, 128L, 192L, 1000L, 1L << 20, 1L << 30})
        for (long y : {1L, 4L, 5L, 192L, 4097L, 1L << 20, 1L << 30})
            for (long z : {1L, 2L, 33L, 192L, 5000L, 1L << 20, 1L << 30}) {
                if (x * y > 1L << 34 || x * y * z > 1L << 34) continue;
                const Geo g{(int)x, (int)y, (int)z, 0, 0, 0, 0.0};
                const int V = x >= 128 ? 2 : 1, cz = norm_chunk(g, V, 4);
                const long cols = (x + 64 * V - 1) / (64 * V) * ((y + 3) / 4), n = cols * ((z + cz - 1) / (long)cz);
                // partials that a context holds or a solve reserves for its points
                const long held = x * y * z / 32 + 65 > 65536 ? x * y * z / 32 + 65 : 65536;
                ++seen;
                if (cols > held || cols >= 1L << 24) continue;  // one chunk in z cannot be fewer blocks
                bad += cz < 2 || n >= 1L << 24 || n > held;
            }
    printf("%ld %ld\n", seen, bad);
    return 0;
}
"""

SHARE = r"""
#include <stdio.h>
#include <vector>
#include "tb7.h"
using namespace gk;

int main() {
    long seen = 0, bad = 0;
    for (int n : {1, 3, 8, 17, 64, 300})
        for (int side : {1, 12, 40, 80, 176})
            for (int rule : {1, 4, 16, 32, 500})
                for (int lay = 0; lay < 4; ++lay) {
                    const bool rb = lay & 1, f64 = lay & 2;
                    std::vector<TBShare> a, b;
                    long tiles = 0;
                    for (int i = 0; i < n; ++i) {
                        const int nz = side + i % 7, cols = (nz + 55) / 56 * ((nz + 23) / 24), own = i % 5 ? rule : 0;
                        a.push_back({cols, nz, own, 0});
                        b.push_back({cols, nz, 0, 0});
                        const int c = own < 1 ? (nz < 16 ? nz : 16) : own < nz ? own : nz;
                        tiles += (long)cols * ((nz + c - 1) / c);
                    }
                    tb_share_chunks(a.data(), n, rb, f64, 4);
                    tb_share_chunks(b.data(), n, rb, f64, 4);
                    for (int i = 0; i < n; ++i) {
                        ++seen;
                        bad += a[i].cz < 1 || a[i].cz > a[i].nz || b[i].cz < 1 || b[i].cz > b[i].nz;
                        const int own = rule < a[i].nz ? rule : a[i].nz;
                        if (tiles >= 512) bad += a[i].cz != (a[i].rule && own > b[i].cz ? own : b[i].cz);
                        else if (a[i].rule) bad += a[i].cz > own;
                    }
                }
    printf("%ld %ld\n", seen, bad);
    return 0;
}
"""

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _run(tmp_path, source):
    src, exe = tmp_path / "rules.hip", tmp_path / "rules"
    src.write_text(source)
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1207_1746_amd", "csrc"), str(src), "-o", str(exe)], check=True,
                   capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return map(int, out.split())


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_admitted_reductions_fit_the_fixed_scratch(tmp_path):
    admitted, over, bad = _run(tmp_path, CHUNKS)
    assert bad == 0
    # the band that is admitted by its count and launches more blocks than the limit is there
    assert admitted > 1000 and over > 0


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_norm_blocks_fit_a_launch(tmp_path):
    seen, bad = _run(tmp_path, NORM)
    assert bad == 0 and seen > 100


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_rules_bound_the_chunks_of_a_batch(tmp_path):
    seen, bad = _run(tmp_path, SHARE)
    assert bad == 0 and seen > 1000
