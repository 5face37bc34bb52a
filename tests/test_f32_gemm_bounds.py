"""Every load of the float32 projections stays inside its row: the kernels' own index arithmetic, compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include "gemm_f32_index.h"
// a row of K floats whose pieces have `piece` k: the loads of every slab that a launch asks for, up to four past the last
static int walk(int K, int piece, int slab) {
    int bad = 0;
    for (int k_first = 0; k_first < K; k_first += piece) {
        const int k = K - k_first < piece ? K - k_first : piece, nk = (k + slab - 1) / slab;
        for (int kt = 0; kt < nk + 4; ++kt)
            for (int chunk = 0; chunk < slab; chunk += 4) {
                const int at = zo2::f32_chunk_at(kt, nk, slab, chunk, k);
                const int want = (kt < nk ? kt : nk - 1) * slab + chunk;
                if (at < 0 || k_first + at + 4 > K || at + 4 > k) ++bad;                                     // past the row, or the piece
                if (zo2::f32_chunk_inside(kt, nk, slab, chunk, k) != (want + 4 <= k) || (want + 4 <= k && at != want)) ++bad;
            }
    }
    return bad;
}
int main() {
    int bad = 0;
    for (int slab = 16; slab <= 32; slab += 16)
        for (int K = 8; K <= 2600; K += 8)
            for (int splits = 1; splits <= 32; ++splits) {
                const int piece = splits == 1 ? K : ((K + splits - 1) / splits + 31) / 32 * 32;
                const int b = walk(K, piece, slab);
                if (b && bad < 20) printf("slab %d K %d piece %d: %d loads\n", slab, K, piece, b);
                bad += b;
            }
    printf("bad %d\n", bad);
    return bad != 0;
}
"""


def test_loads_of_a_slab_past_the_end_of_a_row_stay_inside_it(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2503_12668_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout
