"""CPU test of which way the rules in csrc/gemm_plan.h send the shapes of the GPU tests: a test that is there for one kernel
keeps reaching it when a rule changes, or fails here."""
import heapq
import random
import shutil
import subprocess

import pytest

from paper_2501_02625_amd import _build
from tests import test_gpu_gemm, test_gpu_linear, test_gpu_peft, test_gpu_per_tensor

PROGRAM = r"""
#include <cstdio>
#include "gemm_plan.h"
using namespace halo;

int32_t somewhere;
GemmArgs product(long M, long N, long K) {
    GemmArgs g{};
    g.M = M; g.N = N; g.K = K; g.config = HALO_GEMM_AUTO; g.acc_out = &somewhere;
    return g;
}

// each line: `two M N K` (columns in wide tiles, bf16 out and fp32 out), `one M N K`, `small M N K` (columns of the small tiles), `pair M N K M N K`, `bf16 rows cols pitch` (whole lines?),
// `done n1 t1 n2 t2` (two kinds of tiles, times in tenths), `max rows cols parts` (column maxima reduced first?), // `first log-block rows cols` (stages of the first pass) or `left tokens in out right-block left-block both-products rank`
int main() {
    char what[8];
    while (std::scanf("%7s", what) == 1) {
        long v[7];
        const int count = what[0] == 'o' || what[0] == 's' || what[0] == 'b' || what[0] == 'f' || what[0] == 'm' || what[0] == 't' ? 3 : what[0] == 'd' ? 4 : what[0] == 'p' ? 6 : 7;
        for (int i = 0; i < count; ++i) if (std::scanf("%ld", v + i) != 1) return 1;
        if (what[0] == 'l') {
            GemmArgs gx = product(v[0], v[1], v[2]);
            const GemmArgs gg = product(v[2], v[1], v[0]);
            if (v[6]) { gx.lr_rank = (int)v[6]; gx.acc_out = nullptr; gx.C = &somewhere; gx.c_is_f32 = 1; }
            std::printf("%d\n", (int)left_in_epilogue(gx, v[5] ? &gg : nullptr, (int32_t)v[4], (int32_t)v[3]));
            continue;
        }
        if (what[0] == 'd') {
            std::printf("%.0f\n", 10 * two_kinds_done(v[0], v[1] / 10.0, v[2], v[3] / 10.0));
            continue;
        }
        if (what[0] == 't') {
            GemmArgs g = product(v[0], v[1], v[2]);
            g.transB = 1;
            const long with_sums = (long)two_widths(g);
            g.acc_out = nullptr; g.C = &somewhere;
            std::printf("%ld,%ld\n", (long)two_widths(g), with_sums);
            continue;
        }
        if (what[0] == 'f') {
            std::printf("%d\n", left_first_pass((int)v[0], v[1], v[2]));
            continue;
        }
        if (what[0] == 's') {
            GemmArgs g = product(v[0], v[1], v[2]);
            g.transB = 1;
            std::printf("%d\n", choose_config(g, nullptr) == kSmall32 ? small_tile_columns(g) : 0);
            continue;
        }
        if (what[0] == 'm') {
            std::printf("%d\n", (int)column_maxima_first(v[0], v[1], v[2]));
            continue;
        }
        if (what[0] == 'b') {
            std::printf("%d\n", (int)bf16_whole_lines(v[0], v[1], v[2]));
            continue;
        }
        const GemmArgs a = product(v[0], v[1], v[2]), a2 = product(v[3], v[4], v[5]);
        const int c = choose_config(a, what[0] == 'p' ? &a2 : nullptr);
        std::puts(c == kTiles256 ? "256x256" : c == kTiles256x128 ? "256x128" : c == kTiles128 ? "128x128" : c == kSmall64 ? "64x64"
                  : what[0] == 'o' && a.M <= 16 ? "16x64" : "32x64");
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run([shutil.which("g++") or "g++", "-std=c++17", "-O1", "-I" + _build.CSRC, "-I" + _build.INCLUDE,
                    str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)

    def answers(lines):
        text = "\n".join(" ".join(map(str, l)) for l in lines)
        return subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True).stdout.split()

    return answers


def test_shapes_of_the_small_product_tests(ask):
    shapes, longest = sorted(test_gpu_gemm.SMALL_SHAPES), max(test_gpu_gemm.SMALL_K)
    single = ask(("one", M, N, K) for M, N in shapes for K in test_gpu_gemm.SMALL_K)
    per = len(test_gpu_gemm.SMALL_K)
    for i, s in enumerate(shapes):
        assert set(single[i * per:(i + 1) * per]) == {test_gpu_gemm.SMALL_SHAPES[s][0]}, s
    pairs = ask(("pair", M, N, longest, longest, 48, N // 16 * 16) for M, N in shapes)
    assert dict(zip(shapes, pairs)) == {s: test_gpu_gemm.SMALL_SHAPES[s][1] for s in shapes}


def test_columns_of_the_small_tiles(ask):
    shapes = test_gpu_gemm.NARROW_SHAPES
    assert dict(zip(shapes, map(int, ask(("small", M, N, 4368) for M, N in shapes)))) == shapes
    assert set(ask(("small", M, N, K) for M, N, K, pitch in test_gpu_gemm.ROUND_SHAPES)) == {"32"}


# rows, cols of a dense bf16 output and whether whole lines were the faster store (K = 512, 2 % and more apart, on an MI355X)
WHOLE_LINES = [(288, 4560, False), (6880, 352, False), (1792, 1024, False), (2048, 1024, False), (512, 4096, False),
               (1024, 1056, False), (3072, 1056, False), (512, 2320, False), (2048, 3072, False), (4096, 1536, False),
               (1024, 5120, False), (1536, 4224, False), (1024, 14336, True), (1536, 5120, True), (2048, 4096, True),
               (4096, 2048, True), (8192, 2048, True), (1536, 2320, True), (3072, 2320, True)]


def test_bf16_whole_lines_where_they_are_faster(ask):
    assert ask(("bf16", M, N, N) for M, N, faster in WHOLE_LINES) == [str(int(faster)) for M, N, faster in WHOLE_LINES]
    lines = test_gpu_gemm.LINES
    assert ask(("bf16", M, N, pitch) for M, N, pitch, whole in lines) == [str(int(whole)) for M, N, pitch, whole in lines]


# rows, cols, left block and microseconds of the un-rotation with the first pass taking all stages (eleven at most), eight and
# seven, on an MI355X
FIRST_PASS = [(512, 256, 512, 7.9, 8.8, 8.3), (512, 4096, 512, 13.2, 18.3, 18.1), (1024, 256, 1024, 10.7, 9.8, 9.3),
              (1024, 1024, 1024, 12.6, 13.0, 12.7), (1024, 4096, 1024, 21.0, 26.5, 26.1), (2048, 64, 2048, 16.0, 9.5, 9.4),
              (2048, 256, 2048, 16.3, 10.6, 10.6), (2048, 1024, 2048, 20.8, 18.5, 18.7), (2048, 4096, 2048, 26.6, 34.7, 32.7),
              (4096, 256, 4096, 22.0, 14.0, 14.4), (4096, 1024, 4096, 35.3, 26.4, 28.9), (4096, 4096, 4096, 63.4, 63.5, 59.3),
              (8192, 512, 8192, 34.9, 27.3, 31.6), (8192, 4096, 8192, 126.6, 131.1, 118.9), (4096, 256, 2048, 17.9, 13.5, 13.2),
              (8192, 1024, 2048, 26.8, 33.3, 33.0), (8192, 256, 1024, 16.5, 19.0, 18.7), (16384, 4096, 16384, 284.5, 296.4, 272.4)]


def test_the_first_pass_of_a_left_hand_rotation_is_the_faster_one(ask):
    said = ask(("first", hb.bit_length() - 1, rows, cols) for rows, cols, hb, *us in FIRST_PASS)
    for (rows, cols, hb, whole, eight, seven), stages in zip(FIRST_PASS, said):
        us = {min(hb.bit_length() - 1, 11): whole, 8: eight, 7: seven}
        assert us[int(stages)] <= 1.04 * min(us.values()), (rows, cols, hb, stages)


# tokens, out-features, left block, microseconds of the level-2 backward pass with the column maxima read by every tile and
# reduced first, on an MI355X
COLUMN_MAXIMA = [(960, 4096, 64, 52.9, 55.1), (2112, 1536, 64, 47.4, 48.2), (2112, 14336, 64, 180.7, 178.5), (4160, 4096, 64, 93.7, 86.4),
                 (8128, 512, 64, 78.3, 76.6), (8128, 4096, 64, 189.6, 167.2), (1920, 4096, 128, 54.4, 55.8),
                 (8064, 4096, 128, 164.4, 153.2), (7936, 512, 256, 65.8, 65.7), (8192, 1536, 512, 87.2, 88.2),
                 (8192, 4096, 512, 156.6, 154.9), (8192, 4096, 2048, 166.9, 168.2)]


def test_column_maxima_are_reduced_first_where_that_is_faster(ask):
    said = ask(("max", b, n, b // hb) for b, n, hb, *us in COLUMN_MAXIMA)
    for (b, n, hb, *us), first in zip(COLUMN_MAXIMA, said):
        assert us[int(first)] <= 1.01 * min(us), (b, n, hb)
    assert ask([("max", 8192, 14336, 4), ("max", 8192, 14336, 16)]) == ["0", "1"]      # the launch 4.9 us and 3 saved; 488 us and 478
    lines = test_gpu_linear.MAXIMA          # the first pass takes 64 or 128 rows, or up to 2048 of them
    assert ask(("max", b, n, b // hb) for b, n, hb, first in lines) == [str(int(first)) for b, n, hb, first in lines]


# rows, columns, K and microseconds of a bf16 product in tiles of one width and in the two widths that the rule or a near one takes,
# on an MI355X
TIMED_WIDTHS = [(2048, 14336, 4096, 107.0, 100.0), (2560, 4096, 4096, 46.2, 38.5), (2048, 5120, 4096, 45.4, 36.4),
                (5120, 7296, 4096, 134.5, 112.5), (4608, 5120, 14336, 270.4, 226.0),
                (2896, 3072, 8192, 82.9, 67.4), (816, 10768, 6464, 77.0, 62.0), (1840, 10256, 2432, 49.8, 54.6),
                (4096, 4720, 4096, 74.3, 80.7), (4864, 2256, 1024, 17.8, 19.8), (5888, 1936, 1024, 17.5, 19.4),
                (4096, 4096, 4096, 52.3, 73.2), (8192, 4096, 4096, 104.0, 117.7), (2048, 4096, 4096, 29.5, 35.0)]


def test_tiles_of_two_widths_where_they_are_faster(ask):
    said = [int(s.split(",")[0]) >= 0 for s in ask(("two", M, N, K) for M, N, K, *us in TIMED_WIDTHS)]
    assert said == [one > two for M, N, K, one, two in TIMED_WIDTHS]
    shapes = test_gpu_gemm.TWO_WIDTHS
    assert ask(("two", M, N, K) for M, N, K, *wide in shapes) == ["%d,%d" % (bf16, f32) for M, N, K, bf16, f32 in shapes]


def test_tiles_of_two_kinds_are_done_when_a_dispatch_in_order_is(ask):
    rng = random.Random(5)
    lines = [(rng.randrange(1200), rng.randrange(60, 1600), rng.randrange(1200)) for _ in range(150)] + [(512, 700, 256), (0, 900, 257), (300, 500, 0)]
    lines = [(n1, t1, n2, max(1, round(t1 / rng.uniform(0.4, 1.95)))) for n1, t1, n2 in lines if n1 + n2]
    want = []
    for n1, t1, n2, t2 in lines:
        free = [0] * 256
        for t in [t1] * n1 + [t2] * n2:
            heapq.heapreplace(free, free[0] + t)
        want.append(str(max(free)))
    assert ask(("done", *line) for line in lines) == want


def left(b, m, n, hm, hb, both, rank=0):
    return "left", b, m, n, hm, hb, int(both), rank


def test_shapes_of_the_left_epilogue_tests(ask):
    lines = [left(*s, both=True) for s in test_gpu_linear.LEFT_IN_EPILOGUE]
    lines += [left(b, m, n, min(m & -m, 4096), b & -b, both=False) for b, m, n in test_gpu_per_tensor.LEFT_IN_EPILOGUE]
    lines += [left(b, m, n, hm, hb, both=False, rank=rank) for b, m, n, rank, level, hm, hb in test_gpu_peft.LEFT_IN_EPILOGUE]
    for line, said in zip(lines, ask(lines)):
        assert said == "1", line
    lines = [left(*s, both=True) for s in test_gpu_linear.LEFT_IN_PASSES]
    lines += [left(b, m, n, min(m & -m, 4096), b & -b, both=False) for b, m, n in test_gpu_per_tensor.LEFT_IN_PASSES]
    lines += [left(b, m, n, hm, hb, both=False, rank=rank) for b, m, n, rank, level, hm, hb in test_gpu_peft.LEFT_IN_PASSES]
    for line, said in zip(lines, ask(lines)):
        assert said == "0", line
    # one top stride to five, and none, each on every right block that one kernel finishes or that needs a pass of its own
    tops = {hb.bit_length() - 9 for b, m, n, hm, hb in test_gpu_linear.LEFT_IN_EPILOGUE}
    blocks = {hm for b, m, n, hm, hb in test_gpu_linear.LEFT_IN_EPILOGUE}
    assert tops == {0, 1, 2, 3, 4, 5} and blocks == {512, 1024, 2048, 4096, 3584}


# tokens, in- and out-features, and microseconds of the backward pass of both products with the strides in the epilogue and in
# passes: shapes where the two ways, timed on an MI355X, lie 10 % or more apart
MEASURED = [(256, 1024, 1024, 39.1, 26.1), (256, 8192, 4096, 120.3, 95.8), (512, 8192, 256, 47.2, 41.4), (768, 3072, 1024, 49.4, 42.1),
            (1024, 4096, 4096, 109.2, 96.0), (2048, 1024, 512, 60.8, 51.3), (8192, 2048, 512, 168.2, 147.2),
            (768, 14336, 2048, 136.3, 155.7), (1536, 8192, 64, 62.5, 74.3), (2048, 3072, 1024, 64.9, 74.3),
            (4096, 4096, 4096, 227.1, 256.4), (8192, 14336, 1024, 575.8, 854.0)]


def test_the_faster_way_of_the_left_hand_un_rotation(ask):
    lines = [left(b, m, n, min(m & -m, 4096), b & -b, both=True) for b, m, n, epilogue, passes in MEASURED]
    assert ask(lines) == [str(int(epilogue < passes)) for b, m, n, epilogue, passes in MEASURED]
