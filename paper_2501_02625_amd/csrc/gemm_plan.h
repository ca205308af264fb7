// One INT8 product as its launcher takes it, and the rules that choose between ways to run it: plain host functions, for the
// launchers and for a host program that asks which way a shape goes.
#pragma once
#include <algorithm>
#include <cstdint>

#include "halo.h"

namespace halo {

struct GemmArgs {
    const int8_t* A;
    int64_t lda;
    const int8_t* B;
    int64_t ldb;
    int transB;
    int64_t M, N, K;
    const float* row_scale;
    const float* col_scale;
    void* C;
    int c_is_f32;
    int64_t ldc;
    int32_t* acc_out;
    int64_t ld_acc;
    int config;              // halo_gemm_config: -1 = chosen by shape
    // left_stages == 8 (256-row tiles only, C fp32, M a multiple of 256): the epilogue scales the accumulators,
    // (float(acc) * row_scale[row]) * post_scale[0], and then runs the eight lowest strides (1 .. 128 rows) of a left-hand
    // Walsh-Hadamard rotation down each column of the tile, unnormalised, before it stores C.
    int left_stages;
    const float* post_scale;
    // lr_rank > 0 (C required, no acc_out, N a multiple of 16, not in the small kernel): the epilogue adds a low-rank product
    // to the scaled accumulators before anything else happens to them,
    //   value(row, col) = ((float(acc) * row_scale[row]) * col_scale[col]) * post_scale + sum_k lr_a[row, k] * lr_b[k, col]
    // with lr_a fp32 [M x lr_rank] and lr_b [N x lr_rank] (fp32, or bf16 with lr_b_bf16), both dense, 16-byte aligned,
    // lr_rank a multiple of 8; the sum is accumulated in fp32.
    int lr_rank;
    const float* lr_a;
    const void* lr_b;
    int lr_b_bf16;
    int whole_lines;         // set by the launcher: bf16_whole_lines
};

// bf16 out, tiled kernel: whole 128-byte lines per store request (the trade between lanes is a tenth of the epilogue's
// instructions) or half lines.  Whole ones pay where the stores bind, that is where C outgrows the caches, or where the pieces of
// 64 bytes do not lie on half lines; otherwise the instructions only add up to 0.3 us.  K = 512, half against whole: 1536 x
// 1056 5.7 us / 6.0, 512 x 4096 5.9 / 6.1, 2048 x 3072 8.0 / 8.2, 1536 x 4224 8.1 / 8.2; 1536 x 5120 10.0 / 9.0, 2048 x 4096 10.3 / 9.4,
// 8192 x 2048 17.6 / 14.8; pitch 2320: 512 rows 6.1 / 6.4, 1024 6.6 / 6.5, 1536 7.7 / 6.8, 3072 13.4 / 10.5.
inline bool bf16_whole_lines(int64_t rows, int64_t cols, int64_t pitch) {
    return rows * cols >= (int64_t)(pitch % 32 == 0 ? 7 : 2) << 20;
}

inline int ilog2_exact(int64_t v) {
    int l = 0;
    while ((int64_t(1) << l) < v) ++l;
    return l;
}
inline bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }

// The shapes that launch_row_left_top takes: log_block 9..12 dividing cols, left_top 1..4, or 5 with log_block <= 11, rows a
// multiple of the left block.
inline bool row_left_top_ok(int64_t rows, int64_t cols, int log_block, int left_top) {
    if (log_block < 9 || log_block > 12 || left_top < 1 || left_top > 5) return false;
    if (left_top == 5 && log_block > 11) return false;      // 32 rows of 4096 columns do not fit a compute unit
    if (rows <= 0 || cols <= 0 || cols % (int64_t(1) << log_block) != 0) return false;
    return rows % (int64_t(256) << left_top) == 0;
}

constexpr int64_t kComputeUnits = 256;                            // of a GPU

// Tile configurations (halo_gemm_config in halo.h): 0, 1: 256 x 256; 2: 256 x 128; 3, 4: 128 x 128.  Two more are chosen by
// shape only: 64 x 64 and 32 x 64 (16 x 64) tiles with K split over the wavefronts (gemm_i8_small_kernel).
enum { kTiles256 = 0, kTiles256x128 = 2, kTiles128 = 3, kSmall64 = 5, kSmall32 = 6 };

inline int64_t tiles_of(const GemmArgs& a, int bm, int bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); }
inline double units_of(const GemmArgs& a) { return (double)((a.K + 127) / 128); }

// Estimated microseconds of the tile configurations: so much per tile for the launch of its workgroup, the first loads and the
// store, so much per unit of K.  Two 128 x 128 workgroups share a compute unit, which smooths its last round.
// Coarse: against a kernel trace with warm operands, 28 products from 1024 x 2048 x 512 to 8192 x 4096 x 4096 in each of the
// three tiles, the estimates lie between 27 % below and 47 % above, most of them above and most of all where a round leaves
// compute units idle (256 x 128 tiles at K = 4096: 128 tiles 27.5 us, 256 tiles 31.4, both 34.6 here).  That goes for all three
// tiles alike: the choice is the fastest tile in 26 of the 28 and within 3 % of it in the other two (3072 x 4096 x 4096 with
// sums out: 256 x 256 53.7 us, 128 x 128 52.4).  In tiles of 256 x 256 / 256 x 128 / 128 x 128, bf16 out, 2048 x 4096 x 4096 takes
// 45.3 / 31.4 / 32.9 us, 4096 x 4096 x 4096 52.0 / 60.0 / 62.0, 2048 x 2048 x 2048 25.5 / 16.9 / 12.1.
inline double tile_cost(const GemmArgs& a, int config) {
    const double u = units_of(a), wide = (a.acc_out || a.c_is_f32) ? 4.0 : 0.0;
    if (config == kTiles256) return 8.0 + wide + 1.2 * u;
    if (config == kTiles256x128) return 3.4 + 0.5 * wide + (a.transB ? 0.85 : 0.95) * u;
    return 2.5 + 0.48 * u;
}
inline double product_cost(const GemmArgs& a, int config) {
    const double t = tile_cost(a, config);
    if (config == kTiles128) return 3.0 + std::max(1.0, tiles_of(a, 128, 128) / (double)kComputeUnits) * t;
    const int64_t tiles = config == kTiles256 ? tiles_of(a, 256, 256) : tiles_of(a, 256, 128);
    return 4.0 + (double)((tiles + kComputeUnits - 1) / kComputeUnits) * t;
}
// Tiles of two kinds in one launch, dispatched in order, n1 of the first kind and then n2 of the second: the time at which the last
// one is done, when each compute unit takes the next tile as it gets free.  `late` compute units take one more of the first kind than
// the others, so the second kind's tiles end at f + k t2 on the early ones and at f + t1 + k t2 on the late ones; the first of
// these times at which n2 of them have.  (Times of the late ones count from k = n2 / kComputeUnits on, as when the rules below were
// fitted: where a tile of the first kind takes longer than two of the second, the true one can be earlier.)
inline double two_kinds_done(int64_t n1, double t1, int64_t n2, double t2) {
    const double f = (double)(n1 / kComputeUnits) * t1;           // when the first compute units are free of the first kind
    const int64_t late = n1 % kComputeUnits, early = kComputeUnits - late;
    if (n2 == 0) return f + (late ? t1 : 0.0);
    const int64_t below = (int64_t)(t1 / t2 + 1e-6), above = (int64_t)(t1 / t2 + 1.0 - 1e-6);      // t1 in whole t2
    auto rounds = [](int64_t n, int64_t of) { return n <= 0 ? int64_t(0) : (n + of - 1) / of; };
    int64_t k = rounds(n2, early);                                // if they end before the late ones have done any
    if (k > above) k = rounds(n2 + late * above, kComputeUnits);
    double best = f + (double)k * t2;
    if (late) best = std::min(best, f + t1 + (double)std::max(n2 / kComputeUnits, rounds(n2 - early * below, kComputeUnits)) * t2);
    return std::max(best, f + (late ? t1 : 0.0));
}
// Two products in one launch, the first product's tiles first.
inline double pair_cost(const GemmArgs& a1, const GemmArgs& a2, int config) {
    const double t1 = tile_cost(a1, config), t2 = tile_cost(a2, config);
    if (config == kTiles128) {
        const int64_t n1 = tiles_of(a1, 128, 128), n2 = tiles_of(a2, 128, 128);
        return 3.0 + std::max(std::max(t1, t2), (n1 * t1 + n2 * t2) / kComputeUnits);
    }
    return 4.0 + two_kinds_done(tiles_of(a1, 256, 256), t1, tiles_of(a2, 256, 256), t2);
}

// The configuration of one product, or of a pair (a2).  A product whose 32 x 64 (64 x 64) tiles fit the compute units once
// goes to the small kernel: 16 x 4096 x 4096 4.9 us warm, 7.2 cold (128 x 128 tiles: 15.7, 18), 256 x 1024 x 512 4.3 (6.3),
// 256 x 4096 x 4096 10.3 (16.3), 1024 x 1024 x 1024 6.4 (7.8); at twice as many tiles it is level with the 128 x 128 tiles or
// behind.  A pair takes 128 x 128 tiles where their estimate is 15 % lower: the estimate of a full chip of 128 x 128 tiles is
// too high by about as much as that of a part-filled one of 256 x 256 (measured, 256 x 256 against 128 x 128: two of 4096 x 4096
// x 4096 117 us against 126, 2048 x 4096 x 4096 with its G product 68.9 / 71.6, 3072 x 4096 x 2048 with its G product 71.2 /
// 56.0, 1024 x 4096 x 4096 with its G product 51.7 / 42.6); the faster one on all 14 pairs of that trace.
inline int choose_config(const GemmArgs& a, const GemmArgs* a2) {
    const bool special = a.left_stages || a.lr_rank || (a2 && (a2->left_stages || a2->lr_rank));
    if (!special) {
        if (tiles_of(a, 32, 64) + (a2 ? tiles_of(*a2, 32, 64) : 0) <= kComputeUnits) return kSmall32;
        if (tiles_of(a, 64, 64) + (a2 ? tiles_of(*a2, 64, 64) : 0) <= kComputeUnits) return kSmall64;
    }
    if (a2) return pair_cost(a, *a2, kTiles128) < 0.85 * pair_cost(a, *a2, kTiles256) ? kTiles128 : kTiles256;
    int best = kTiles256;
    for (const int c : {kTiles256x128, kTiles128})
        if (product_cost(a, c) < product_cost(a, best)) best = c;
    return best;
}

// Tiles of two widths in one launch (one product, K-contiguous B): the first `wide` columns in tiles of 256 x 256, the others in
// 256 x 192, so that the last round fills the compute units or is a shorter one.  Returns `wide` where that is the faster way by
// estimate, otherwise -1.  The estimate of a narrow tile where all run at once and where they do not, and how far that of the 128 x 128
// tiles is above what they take there, are fitted to 180 products, sizes drawn over 256 .. 8192 by 256 .. 14336 by 256 .. 14336, timed
// in one width and in two: those that go in two widths gain 10 % in the mean, the worst loses 3 % (2992 x 8192 x 4352, fp32 out).  bf16 out, one width / two:
// 2560 x 4096 x 4096 46.2 us / 38.5, 2048 x 5120 x 4096 45.4 / 36.4, 2896 x 3072 x 8192 82.9 / 67.4, 5120 x 7296 x 4096 134.5 / 112.5,
// 4608 x 5120 x 14336 270 / 226, 6112 x 14336 x 832 124.5 / 126.1 (not taken); fp32 out 2048 x 14336 x 4096 115.7 / 105.6.  (224 columns
// fill 2048 x 14336 in two equal rounds, but a bf16 row of a tile is then no whole number of cache lines: 118 us against 107 with 256.)
// The search runs on the host before every such launch: 0.5 us at 14336 columns, 2 at 128256, 0.02 where 4096 by 4096 fit once.
inline int64_t two_widths(const GemmArgs& a) {
    if (a.config >= 0 || a.left_stages || a.lr_rank || a.N % 16 != 0 || !a.transB) return -1;
    const int c = choose_config(a, nullptr);
    if (c == kSmall32 || c == kSmall64) return -1;
    const int64_t panels = (a.M + 255) / 256;
    const double u = units_of(a), wide_out = (a.acc_out || a.c_is_f32) ? 3.0 : 0.0, one_width = product_cost(a, c);
    const double wide_tile = tile_cost(a, kTiles256), narrow_tile = 7.0 + wide_out + 0.95 * u;
    double best = 1e30;
    int64_t wide = -1;
    for (int64_t n1 = 0; n1 * 256 < a.N; ++n1) {
        const int64_t n2 = (a.N - n1 * 256 + 191) / 192;
        const bool at_once = panels * (n1 + n2) <= kComputeUnits;
        if (at_once && n1 > 0) continue;
        const double limit = one_width * (c != kTiles128 ? 1.0 : !at_once ? 0.88 : u < 12 ? 0.85 : 0.92);
        // no split is done before all compute units have shared its work evenly: most are out without the estimate
        const double evenly = (double)panels * ((double)n1 * wide_tile + (double)n2 * narrow_tile) / (double)kComputeUnits;
        if (!at_once && 4.0 + evenly > std::min(best, limit) + 1e-3) continue;
        const double t = 4.0 + (at_once ? wide_out + 8.5 + 0.84 * u : two_kinds_done(panels * n1, wide_tile, panels * n2, narrow_tile));
        if (t < limit && t < best) {
            best = t;
            wide = n1 * 256;
        }
    }
    return wide;
}

// Columns of the small kernel's tiles of 16 and 32 rows (kSmall32), one product with a K-contiguous B: 16 or 32 instead of 64 while
// all tiles still run at once, one per compute unit.  There the rate at which B arrives is the bound, and every compute unit has to
// fetch; narrow tiles also leave room for more ring stages.  They read A two or four times as often, which stays in the caches.
// 64 columns against the narrow tile, B from memory: 16 x 4096 x 4096 9.8 us / 7.2, 16 x 4096 x 14336 25.8 / 14.8, 32 x 4096 x
// 4096 10.8 / 8.0, 64 x 4096 x 4096 10.9 / 8.9, 128 x 2048 x 4096 7.8 / 6.5, 16 x 8192 x 4096 11.2 / 10.5.  With B in the caches:
// 16 x 4096 x 4096 5.4 / 4.9, 32 x 4096 x 4096 6.5 / 6.1, 128 x 2048 x 4096 6.5 / 5.9, 16 x 8192 x 4096 6.6 / 6.3; of 176 shapes, 16 .. 128
// rows by 1024 .. 14336 by 2048 .. 14336, each both ways, 64 x 4096 x 4096 alone is more than 2 % slower, 6.7 / 7.0; of others tried, 16 x 8192 x 8064 (12.8 / 13.5; from
// memory 17.6 / 14.7).
inline int small_tile_columns(const GemmArgs& a) {
    if (!a.transB) return 64;
    const int rows = a.M <= 16 ? 16 : 32;
    return tiles_of(a, rows, 16) <= kComputeUnits ? 16 : tiles_of(a, rows, 32) <= kComputeUnits ? 32 : 64;
}

// Estimated microseconds of launch_gemm_i8(a) / launch_gemm_i8_pair(a, *a2), for choices between ways to split the work.
inline double gemm_i8_cost(const GemmArgs& a, const GemmArgs* a2) {
    const int c = a.config < 0 ? choose_config(a, a2) : a.config;
    // 64 columns: 16 x 512 x 512 3.9 us, 256 x 1024 x 2048 5.5, 256 x 4096 x 4096 10.3 and 13.8 with a K-strided B.  Narrow tiles
    // are not in it: a product with a K-contiguous B has no other way than one launch.
    if (c == kSmall32 || c == kSmall64) return 3.5 + 0.8 * units_of(a) / 4 + (a2 ? 0.8 * units_of(*a2) / 4 : 0.0);
    const double t = a2 ? pair_cost(a, *a2, c) : product_cost(a, c);
    if (!a.left_stages && !(a2 && a2->left_stages)) return t;
    // what the left-hand epilogue adds (5 to 6 us with 128 and 384 tiles in the launch, 17 with 512), over an estimate that is
    // high where the chip is not full
    const double fill = (double)(tiles_of(a, 256, 256) + (a2 ? tiles_of(*a2, 256, 256) : 0)) / kComputeUnits;
    return t + 3.0 + 4.0 * std::min(1.0, fill);
}

// Stages, from stride 1 on, that one pass over blocks of rows takes at most.
constexpr int kColBlockStages = 11;
// Stages of the first pass of a left-hand rotation that runs all of its strides in passes of its own (log_block >= 7): all of
// them where that pass alone fills the chip enough; otherwise seven or eight, which many small workgroups run, and a strided pass
// for the rest.  A workgroup of the first pass holds 2^stages rows of 32 columns, so with eleven stages 2048 x 1024 is 32 of them.
// Un-rotation of int32, rows x cols of one block, all stages (or eleven) in the first pass / eight / seven: 1024 x 256 10.7 us / 9.8
// / 9.3, 1024 x 1024 12.6 / 13.0 / 12.7, 1024 x 4096 21.0 / 26.5 / 26.1, 2048 x 256 16.3 / 10.6 / 10.6, 2048 x 1024 20.8 / 18.5 /
// 18.7, 2048 x 4096 26.6 / 34.7 / 32.7, 4096 x 1024 35.3 / 26.4 / 28.9, 8192 x 256 27.7 / 20.0 / 23.9, 4096 x 4096 63.4 / 63.5 / 59.3,
// 8192 x 4096 127 / 131 / 119, 16384 x 4096 285 / 296 / 272.
inline int left_first_pass(int log_block, int64_t rows, int64_t cols) {
    if (log_block <= 9 || (log_block <= kColBlockStages && (((cols + 31) / 32) * (rows >> log_block)) >> (log_block - 5) > 0))
        return log_block;
    const bool large = rows * cols >= (int64_t(1) << 24);
    return std::max(large || log_block <= kColBlockStages ? 7 : 8, log_block - (large ? 7 : 6));
}

// The transposed column quantiser behind a left-hand rotation, whose first pass leaves a vector of the columns' maxima per block
// of rows: every tile (128 x 128) reads the vectors of its columns, or one launch more reduces them first.  The launch costs 1 to 2
// us, the reading some 6 TB/s from the second-level caches.  Level-2 backward, 256 in-features, tokens x out-features and vectors,
// read by every tile / reduced first: 2112 x 1536, 33 47.4 us / 48.2, 4160 x 512, 65 57.6 / 57.6, 4160 x 4096 93.7 / 86.4, 8128 x 4096,
// 127 189.6 / 167.2 (169.3 with atomic maxima), 8192 x 4096, 16 156.6 / 154.9, 8192 x 4096, 4 166.9 / 168.2.  A few
// vectors are next to nothing beside a tile: at 8192 x 14336, 4 the launch takes 4.9 us and saves 3, with 8 both ways take 490.
inline bool column_maxima_first(int64_t rows, int64_t cols, int64_t parts) {
    return parts > 8 && ((rows + 127) / 128) * ((cols + 127) / 128) * parts * 512 > (int64_t(10) << 20);
}

// Level 2: the low eight strides of the left-hand un-rotation of E_X can run in the epilogue of the E product when the
// left block covers whole 256-row tiles.  They do when that is the faster way: a small product is better off in smaller
// tiles, followed by one pass over its accumulators or two (left_first_pass).  gx, gg: the plain forms of the products (gg null: only
// E_X is wanted).  Microseconds, fitted to the measurement below: half of the difference between the products' estimates (which are
// high where the chip is not full); 4 for the epilogue, and 1 per million elements for a strided pass behind it where no one kernel
// finishes; for the passes 1 per million elements, 2 beyond 30 million (the caches), 5.5 where the first one starts from int32
// accumulators, 3.5 where it takes eleven strides, 2.5 and 0.5 per million elements for a second one.
// The backward pass timed both ways on 379 shapes, 256 .. 8192 tokens, 512 .. 14336 by 64 .. 4096, each with both products, with E_X
// alone and with rank-16 adapters: the rule takes the faster way or one within 3 % of it in 1102 of 1137; five are more than 10 %
// behind, 17 % at worst (1536 x 5632 by 64, E_X and G, 54 us in the epilogue and 63 in passes).  Both products, in the epilogue against
// passes: 256 x 8192 x 4096 120 us / 96, 1024 x 4096 x 4096 109 / 96, 512 x 8192 x 256 47 / 41, 4096 x 2048 x 1024 92 / 90, 2048 x 3072 x
// 1024 65 / 74, 4096 x 4096 x 4096 227 / 256, 8192 x 14336 x 1024 576 / 854.
inline bool left_in_epilogue(const GemmArgs& gx, const GemmArgs* gg, int32_t hb, int32_t hm) {
    const int64_t b = gx.M, m = gx.N;
    if (hb < 256 || b % 256) return false;
    GemmArgs l = gx, g2 = gg ? *gg : gx;
    l.left_stages = 8; l.config = HALO_GEMM_256x256x64; g2.config = HALO_GEMM_256x256x64;
    const int stages = ilog2_exact(hb), top = stages - 8;
    const bool one_kernel = is_pow2(hm) && row_left_top_ok(b, m, ilog2_exact(hm), top);
    const bool second = left_first_pass(stages, b, m) < stages;
    const double melems = (double)b * (double)m / 1e6;
    const double products = 0.5 * (gemm_i8_cost(l, gg ? &g2 : nullptr) - gemm_i8_cost(gx, gg));
    const double epilogue = 4.0 + (top == 0 || one_kernel ? 0.0 : melems);
    const double passes = melems + std::max(0.0, melems - 30.0) + (gx.lr_rank ? 0.0 : 5.5) +
                          (second ? 2.5 + 0.5 * melems : stages == kColBlockStages ? 3.5 : 0.0);
    return products + epilogue <= passes;
}

}  // namespace halo
