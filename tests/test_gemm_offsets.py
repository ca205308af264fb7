"""CPU test of the addresses that the INT8 GEMM kernels fetch a K-strided B from (csrc/gemm_offsets.h).

B may be a column slice of a wider matrix: its last row then ends at the end of the allocation, before its pitch does.  A host
program, compiled from the kernels' own header, walks every request of every tile and reports the furthest byte that is
fetched, and whether every column of the matrix was."""
import shutil
import subprocess

import pytest

from paper_2501_02625_amd import _build

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "gemm_offsets.h"
using namespace halo;

// WAVES wavefronts of REQUESTS requests fetch the 128 rows of a unit.  Furthest byte past the start of the unit's last row.
template <int BN, int WAVES, int REQUESTS>
bool walk(int64_t N, int64_t ldb, int64_t room) {
    typedef KMajorRequests<BN> R;
    std::vector<char> seen((N + 15) / 16 * 16);
    int64_t furthest = 0;
    for (int64_t n0 = 0; n0 < N; n0 += BN)
        for (int wave = 0; wave < WAVES; ++wave)
            for (int lane = 0; lane < 64; ++lane)
                for (int i = 0; i < REQUESTS; ++i) {
                    const int row = R::first_row(wave, lane, REQUESTS) + i * R::ROWS;
                    if (row > 127) return false;
                    const uint32_t off = R::offset(row, R::column(lane, i), ldb, R::columns(N, n0));
                    if (off == kOutside) continue;
                    const int64_t at = n0 + off - (int64_t)row * ldb;      // column of the matrix, on a row that may be the last
                    furthest = std::max(furthest, at + 16);
                    if (row == 127) for (int b = 0; b < 16; ++b) if (at + b < (int64_t)seen.size()) seen[at + b] = 1;
                }
    bool all = true;
    for (int64_t c = 0; c < N; ++c) all = all && seen[c];
    if (furthest > room || !all)
        std::printf("BN %d N %ld ldb %ld: fetches to byte %ld of a last row with %ld, all columns %d\n", BN, (long)N, (long)ldb,
                    (long)furthest, (long)room, (int)all);
    return furthest <= room && all;
}

int main() {
    bool ok = true;
    for (int64_t N : {1, 16, 40, 48, 64, 72, 112, 128, 144, 250, 256, 272, 500})
        for (int64_t c0 : {0, 16, 64, 240, 1024})                          // first column of the slice
            for (int64_t behind : {0, 16, 256}) {                          // columns of the wide matrix after it
                const int64_t padded = (N + 15) / 16 * 16, ldb = c0 + padded + behind;
                const int64_t room = ldb - c0;                             // bytes from the last row's start to the end
                ok = walk<256, 4, 8>(N, ldb, room) && ok;
                ok = walk<128, 4, 4>(N, ldb, room) && ok;
                ok = walk<64, 1, 8>(N, ldb, room) && ok;
            }
    return ok ? 0 : 1;
}
"""


def test_no_request_reaches_past_the_last_row(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", _build.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
