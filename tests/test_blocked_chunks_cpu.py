"""Host rules of a blocked pass's launch (compiled here for the host alone): the
z chunk it takes, and the count that decides whether its fused reduction fits
the fixed scratch of gscl_do_all_noalloc.  Every admitted call has at most as
many blocks as the scratch holds, around the limit, for every number of levels
and both layouts, with the chunk picked and with one set."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
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


@pytest.mark.skipif(not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")), reason="no hipcc")
def test_admitted_reductions_fit_the_fixed_scratch(tmp_path):
    src, exe = tmp_path / "chunks.hip", tmp_path / "chunks"
    src.write_text(SOURCE)
    subprocess.run([shutil.which("hipcc") or "/opt/rocm/bin/hipcc", "--offload-host-only", "-std=c++17", "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1207_1746_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    admitted, over, bad = map(int, out.split())
    assert bad == 0
    # the band that is admitted by its count and launches more blocks than the limit is there
    assert admitted > 1000 and over > 0
