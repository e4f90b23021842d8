"""The rows that the semi-join's mask kernel loads, walked on the CPU with the
arithmetic the kernel and its launcher use (csrc/semirows.hpp): every load of every
form lies inside the table, for short tables and for short last parts alike."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2209_04579_amd", "csrc")

WALK = r"""
#include <initializer_list>
#include <stdio.h>
#include "semirows.hpp"
using namespace tqp;

// The first key beyond the `rows` rows that a launch over them loads, or -1.  Chunks from
// the first on, and some past the end (a wave loads its next chunk before it
// knows that there is none).
template <int V> static int64_t beyond(int64_t rows, bool aligned, int64_t first) {
    const int64_t chunks = (rows + kSjChunk - 1) / kSjChunk + 40;
    for (int64_t c = first; c < chunks; c++) {
        const int64_t row0 = c * kSjChunk;
        for (uint32_t lane = 0; lane < 64; lane++) {
            if (sj_whole_chunks(aligned, rows)) {
                const int64_t at = sj_chunk_row(row0, rows);
                for (int k = 0; k < kSjIPT / V; k++) {
                    const int64_t key = at + sj_lane_key<V>(lane, k);
                    if (key % V != 0) return key;
                    if (key + V > rows) return key + V - 1;
                }
            }
            if (row0 < rows)
                for (int r = 0; r < kSjIPT; r++) {
                    const int64_t key = row0 + sj_any_row(row0, rows, lane, r);
                    if (key < row0 || key >= rows) return key;
                }
        }
    }
    return -1;
}

static int check(int64_t n, int64_t most) {
    for (int64_t row0 = 0; row0 < n;) {
        const int64_t rows = sj_part_rows(n, row0, most);
        if (rows < 1 || rows > most) { printf("part of %lld rows\n", (long long)rows); return 1; }
        const int64_t first = rows > 100 * kSjChunk ? rows / kSjChunk - 50 : 0;
        for (int aligned = 0; aligned < 2; aligned++) {
            const int64_t a = beyond<4>(rows, aligned, first), b = beyond<2>(rows, aligned, first);
            if (a >= 0 || b >= 0) {
                printf("n %lld, part at %lld of %lld rows, aligned %d: loads key %lld\n", (long long)n,
                       (long long)row0, (long long)rows, aligned, (long long)(a >= 0 ? a : b));
                return 1;
            }
        }
        row0 += rows;
    }
    return 0;
}

int main() {
    int bad = 0;
    for (int64_t n = 1; n <= 1100 && bad < 5; n++) bad += check(n, n);
    for (int64_t r : {1, 2, 3, 4, 7, 8, 64, 255, 510, 511, 512, 513, 1000, 1024})
        for (int parts = 1; parts <= 2; parts++) bad += check(parts * kSjPartRows + r, kSjPartRows);
    // an aligned table of whole chunks is loaded as such
    if (!sj_whole_chunks(true, kSjChunk) || sj_whole_chunks(false, kSjChunk)) bad++;
    return bad ? 1 : 0;
}
"""


def test_every_load_is_inside_the_table(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
