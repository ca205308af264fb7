// INT8 GEMM on the CDNA4 matrix cores (v_mfma_i32_16x16x64_i8) with int32 accumulation and a fused
// dequantisation epilogue:  C = diag(row_scale) * (A * op(B)) * diag(col_scale).
//
//   A  [M x K]  K contiguous.
//   B  transB:  [N x K], K contiguous.
//      !transB: [K x N], K strided: the saved (WH)_Q / (XH)_Q codes are reused by the backward products as they are,
//               without a transposed copy in HBM.
//
// What bounds it, and what the design follows from.  On real codes the chip is limited by power, not by issue slots: a
// loop of nothing but matrix instructions on Gaussian codes runs at 3.45 POP/s with v_mfma_i32_32x32x32_i8, 4.15 with
// v_mfma_i32_16x16x64_i8 (half the accumulator traffic per operation), and 4.3 when two instructions in a row add to the
// same accumulator; all three reach 4.9 on zeros.  LDS reads cost little on top, the global->LDS stream about a quarter.
// Hence: the 16x16x64 instruction, K taken 128 bytes at a time with the two instructions of an accumulator back to back,
// four wavefronts of 128 x 128 (one per SIMD, 256 accumulators in AGPRs) instead of eight of 128 x 64 (a third fewer LDS
// reads), and the largest tile the register file holds.  4096 x 4096 x 14336, fp32 out: 157 us (3.07 POP/s); the previous
// kernel, eight wavefronts on 32x32x32, took 205.  The main loop issues a matrix instruction every 16.6 cycles (16 is the
// pipe's rate) and the clock settles at 1.7 GHz on such operands.
//
// Main loop.  Workgroup = 2 x 2 wavefronts, each a grid of TM x TN tiles of 16 x 16; one UNIT = 128 bytes of K.  A sits in
// a ring of three LDS stages, B in a ring of two, filled by buffer_load_dwordx4 ... lds (global memory -> LDS without passing
// through registers): in unit u the A stage of unit u+3 and the B stage of unit u+2 are requested.  Fragments: all of B's
// of the next unit are read during this one (two register sets), A's are read in place as soon as the last matrix
// instruction of their row is issued.  One barrier per unit, after its first row of tiles: by then the wavefront holds all
// fragments of this unit (so its stages may be overwritten) and has waited for its share of the next unit's stages.  All of
// it is inline assembly in program order: the compiler would order every LDS read after every outstanding global->LDS
// transfer, and the order of the instructions is the schedule.  Other instructions go between accumulator pairs only.
// What lies beyond the matrix, in rows, columns or K: those lanes of a request get an offset past the end of the buffer
// descriptor (kOutside), for which the hardware writes zeros to LDS and touches no memory.  Rows and columns are decided once
// per tile, K when the last stage is reached (trim_a, trim_b).
// A launch may carry two independent products (halo_gemm_i8_pair): workgroups past the first product's tile count take the
// second argument block.
//
// Operand layout (16x16x64 i8): lane l supplies 16 consecutive K-bytes of row (l % 16), from K offset 16 * (l / 16) of the
// 64-byte step.  B is passed as the instruction's first operand and A as its second, so a lane ends up with FOUR CONSECUTIVE
// COLUMNS of one row of C: row l % 16, columns 4 * (l / 16) .. + 3 of the tile, and the stores need no staging through LDS.
//
// LDS layouts.  K-contiguous operands: rows of 128 bytes, the 16-byte chunk index XOR-swizzled with (row / 2) % 8: the 16
// rows that a quarter of a wavefront reads fall in 16 different bank groups.  A DMA lane writes LDS slot (slot base + lane),
// so the swizzle is applied to the global address it fetches; a request covers whole 128-byte lines.  K-strided B: stored as
// it lies in memory (K-major rows of BN bytes) and transposed by the LDS read itself, ds_read_b64_tr_b8: a group of 16 lanes
// reads an 8(k) x 16(n) byte block, lane i supplying the address of row i/2, half i%2, and receiving column i; the two
// groups of a half-wavefront read rows 0-7 and 16-23, which the swizzle (kmajor_swizzle) spreads over all banks.
#include <algorithm>
#include <mutex>

#include "gemm_offsets.h"
#include "halo_internal.h"
#include "matrix_asm.h"

namespace halo {
namespace {

template <int TM_, int TN_, bool TRANSB>
struct GemmCfg {
    static constexpr int TM = TM_, TN = TN_;                     // 16 x 16 tiles per wavefront
    static constexpr int WM = 16 * TM, WN = 16 * TN;
    static constexpr int BM = 2 * WM, BN = 2 * WN;               // macro tile
    static constexpr int BK = 128;                               // K bytes per unit
    static constexpr int NT = 256;
    // tile-rows per group of the workgroup->tile map (4 measured best of 2/4/8/16 on the Llama-shaped products)
    static constexpr int GROUP_M = 4;
    static constexpr int NSA = 3, NSB = 2;                       // ring stages
    static constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK;
    static constexpr int LA = A_BYTES / 4096, LB = B_BYTES / 4096;   // DMA instructions per wavefront and stage
    static constexpr int LDS_BYTES = NSA * A_BYTES + NSB * B_BYTES;
    static constexpr int ROW = 2 * TN;                           // matrix instructions per row of tiles
    // TN a multiple of 4: a wavefront's columns lie together.  Six column tiles (192 columns): four together and, behind all of those,
    // two, so that the whole lines that the epilogue stores start at a line.
    static constexpr int LOW_STEP = TN % 4 ? TN - 2 : TN;        // column tiles between the two wavefronts' first ones
    static __device__ __forceinline__ int high_column(int wave_n) { return 16 * (2 * LOW_STEP + 2 * wave_n); }
    static_assert(TN % 4 == 0 || (TN % 4 == 2 && TRANSB), "column tiles");
    static constexpr int READS_B = TRANSB ? 2 * TN : 4 * TN;     // LDS read instructions for B's fragments of one unit
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

template <int OFF>
__device__ __forceinline__ void lds_read16(v4i& d, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void lds_read8_tr(v2i& d, uint32_t addr) {
    asm volatile("ds_read_b64_tr_b8 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
template <int T>
__device__ __forceinline__ void mfma(const v4i& b, const v4i& a) {
    asm volatile("v_mfma_i32_16x16x64_i8 a[%2:%3], %0, %1, a[%2:%3]" ::"v"(b), "v"(a), "n"(4 * T), "n"(4 * T + 3));
}
// Row of a 16-row tile that lane l % 16 works on.  A linear renumbering in which the rows that a stride of 4 pairs sit in
// lanes l and l ^ 7, so that each of the strides 1, 2, 4, 8 (lane masks 1, 2, 7, 8) is one DPP operand.
__device__ __forceinline__ int row_of_lane(int l16) { return (l16 & 4) ? l16 ^ 3 : l16; }

// Where the accumulators of a lane lie in C.  Register tile (i, j) holds row row0 + 16 i and the four columns from
// col(j); the first and the second half of the column tiles have their own base: with SWAP, the two wavefronts that share
// columns hold the halves in opposite order (epilogue_left8).  192-column tiles: GemmCfg::high_column.
template <class Cfg>
struct Place {
    int64_t row0, col_lo, col_hi;
    static constexpr int LOW = Cfg::TN % 4 ? Cfg::TN - 2 : Cfg::TN / 2;      // column tiles of the first part
    __device__ __forceinline__ Place(int64_t m0, int64_t n0, int wave, int lane, bool swap) {
        const int wave_m = wave >> 1, wave_n = wave & 1;
        row0 = m0 + wave_m * Cfg::WM + row_of_lane(lane & 15);
        const int64_t c = n0 + wave_n * 16 * Cfg::LOW_STEP + 4 * (lane >> 4);
        const bool s = swap && wave_m;
        col_lo = c + (s ? Cfg::WN / 2 : 0);
        col_hi = Cfg::TN % 4 ? n0 + Cfg::high_column(wave_n) + 4 * (lane >> 4) : c + (s ? 0 : Cfg::WN / 2);
    }
    __device__ __forceinline__ int64_t col(int j) const { return j < LOW ? col_lo + 16 * j : col_hi + 16 * (j - LOW); }
};

// Register fragments of one wavefront: A's of the current unit (replaced row by row), B's of this unit and the next; bt are
// the halves of B's fragments as the transposing reads deliver them.
template <class Cfg>
struct Frags {
    v4i a[2][Cfg::TM];
    v4i b[2][2][Cfg::TN];
    v2i bt[2][2][Cfg::TN][2];
};

// The main loop of one tile: fills the accumulators.  m0, n0: the tile's first row and column.
template <class Cfg, bool TRANSB, bool SWAP>
__device__ __forceinline__ void main_loop(const GemmArgs& a, int64_t m0, int64_t n0, int wave, int lane, unsigned char* smem) {
    constexpr int TM = Cfg::TM, TN = Cfg::TN, BK = Cfg::BK, BN = Cfg::BN, LA = Cfg::LA, LB = Cfg::LB;
    using KMajor = KMajorRequests<BN>;
    constexpr int RPI = KMajor::ROWS;
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const int l16 = lane & 15, g4 = lane >> 4, lrow = row_of_lane(l16);
    const int units = (int)((a.K + BK - 1) / BK);
    const uint32_t lds_a = (uint32_t)(uintptr_t)HALO_LDS_PTR(smem);
    const uint32_t lds_b = lds_a + Cfg::NSA * Cfg::A_BYTES;

    // ---- source offsets of this lane's DMA requests, relative to the tile's first row / column at the stage's first K.
    // Rows and columns beyond the matrix (columns in whole chunks) come as zeros.
    // K-contiguous operand: request i covers rows 8 i .. of this wavefront's share; their swizzle differs by bit 2 of the
    // chunk between even and odd i.  ka[i & 1]: K offset of the lane's chunk.
    uint32_t avo[LA], bvo[LB];
    const int r8 = lane >> 3;
    const int k0 = 16 * ((lane & 7) ^ (r8 >> 1));
    const int kc[2] = {k0, k0 ^ 64};
    const int64_t rows_a = a.M - m0, rows_b = a.N - n0, cols_b = KMajor::columns(a.N, n0);
    {
        const int row = wave * LA * 8 + r8;
        const uint32_t off = (uint32_t)row * (uint32_t)a.lda;
#pragma unroll
        for (int i = 0; i < LA; ++i)
            avo[i] = row + 8 * i < rows_a ? off + (uint32_t)(8 * i) * (uint32_t)a.lda + kc[i & 1] : kOutside;
    }
    const int krow = TRANSB ? 0 : KMajor::first_row(wave, lane, LB);   // K-strided B: this lane's first K-major row
    if constexpr (TRANSB) {
        const int row = wave * LB * 8 + r8;
        const uint32_t off = (uint32_t)row * (uint32_t)a.ldb;
#pragma unroll
        for (int i = 0; i < LB; ++i)
            bvo[i] = row + 8 * i < rows_b ? off + (uint32_t)(8 * i) * (uint32_t)a.ldb + kc[i & 1] : kOutside;
    } else {
#pragma unroll
        for (int i = 0; i < LB; ++i) bvo[i] = KMajor::offset(krow + i * RPI, KMajor::column(lane, i), a.ldb, cols_b);
    }
    v4u abuf = make_buffer(a.A + m0 * a.lda), bbuf = make_buffer(TRANSB ? a.B + n0 * a.ldb : a.B + n0);
    const int64_t b_step = TRANSB ? (int64_t)BK : (int64_t)BK * a.ldb;
    // left_a / left_b: K bytes from the stage that the offsets stand for to the end.  What lies beyond K is not fetched.
    int64_t left_a = a.K, left_b = a.K;
    auto trim_a = [&]() {
#pragma unroll
        for (int i = 0; i < LA; ++i) avo[i] = kc[i & 1] < left_a ? avo[i] : kOutside;
    };
    auto trim_b = [&]() {
#pragma unroll
        for (int i = 0; i < LB; ++i) bvo[i] = (TRANSB ? kc[i & 1] : krow + i * RPI) < left_b ? bvo[i] : kOutside;
    };
    auto dma_a = [&](int slot, int i) { dma16(avo[i], abuf, lds_a + slot * Cfg::A_BYTES + (wave * LA + i) * 1024); };
    auto dma_b = [&](int slot, int i) { dma16(bvo[i], bbuf, lds_b + slot * Cfg::B_BYTES + (wave * LB + i) * 1024); };
    auto next_a = [&]() {
        advance(abuf, BK);
        left_a -= BK;
        if (left_a < BK) trim_a();
    };
    auto next_b = [&]() {
        advance(bbuf, b_step);
        left_b -= BK;
        if (left_b < BK) trim_b();
    };
    if (left_a < BK) {
        trim_a();
        trim_b();
    }
    // ---- first stages, in the order in which they are needed
#pragma unroll
    for (int i = 0; i < LA; ++i) dma_a(0, i);
#pragma unroll
    for (int i = 0; i < LB; ++i) dma_b(0, i);
    next_a();
    next_b();
#pragma unroll
    for (int i = 0; i < LB; ++i) dma_b(1, i);
#pragma unroll
    for (int i = 0; i < LA; ++i) dma_a(1, i);
    next_a();
    next_b();
#pragma unroll
    for (int i = 0; i < LA; ++i) dma_a(2, i);
    next_a();
    // ---- clear the accumulators while the first stages are on their way
    hold_accumulators<TM * TN>();
    StaticFor<0, TM * TN>::run([&](auto t) { clear_acc<decltype(t)::value>(); });
    // ---- fragment addresses inside stage 0 (for K-strided B the K half and the second row block are immediate offsets)
    uint32_t a_addr[2], b_addr[TRANSB ? 2 : TN], b_high[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) a_addr[k] = lds_a + (wave_m * Cfg::WM + lrow) * BK + 16 * ((4 * k + g4) ^ (lrow >> 1));
    if constexpr (TRANSB) {
        static_assert(!SWAP, "the left-hand epilogue is for K-strided B");
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            b_addr[k] = lds_b + (wave_n * 16 * Cfg::LOW_STEP + l16) * BK + 16 * ((4 * k + g4) ^ (l16 >> 1));
            b_high[k] = lds_b + (Cfg::high_column(wave_n) + l16) * BK + 16 * ((4 * k + g4) ^ (l16 >> 1));
        }
    } else {
        const int row = 16 * g4 + (l16 >> 1);
        const int turn = kmajor_swizzle<BN>(row) ^ (wave_n * TN) ^ (SWAP && wave_m ? TN / 2 : 0);
#pragma unroll
        for (int j = 0; j < TN; ++j) b_addr[j] = lds_b + row * BN + 16 * (j ^ turn) + 8 * (l16 & 1);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LA + LB) : "memory");
    asm volatile("s_barrier" ::: "memory");
    Frags<Cfg> f;
    auto read_a = [&](auto ii, auto kk, uint32_t stage) {
        constexpr int i = decltype(ii)::value, k = decltype(kk)::value;
        lds_read16<i * 16 * BK>(f.a[k][i], a_addr[k] + stage);
    };
    auto read_b = [&](auto ss, auto qq, uint32_t stage) {
        constexpr int s = decltype(ss)::value, q = decltype(qq)::value;
        if constexpr (TRANSB) {
            constexpr int k = q & 1, j = q >> 1;
            if constexpr (TN % 4 && j >= Cfg::LOW_STEP) lds_read16<(j - Cfg::LOW_STEP) * 16 * BK>(f.b[s][k][j], b_high[k] + stage);
            else lds_read16<j * 16 * BK>(f.b[s][k][j], b_addr[k] + stage);
        } else {
            constexpr int h = q & 1, k = (q >> 1) & 1, j = q >> 2;
            lds_read8_tr<k * 64 * BN + h * 8 * BN>(f.bt[s][k][j][h], b_addr[j] + stage);
        }
    };
    // The registers that a wait has made valid, passed through empty assembly so that nothing that uses them moves above it.
    auto settle_b = [&](auto ss) {
        constexpr int s = decltype(ss)::value;
        auto& fb = f.b;
        auto& ft = f.bt;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (TRANSB) {
                    asm volatile("" : "+v"(fb[s][k][j]));
                } else {
                    asm volatile("" : "+v"(ft[s][k][j][0]), "+v"(ft[s][k][j][1]));
                    fb[s][k][j] = (v4i){ft[s][k][j][0][0], ft[s][k][j][0][1], ft[s][k][j][1][0], ft[s][k][j][1][1]};
                }
            }
    };
    StaticFor<0, Cfg::READS_B>::run([&](auto q) { read_b(Int<0>(), q, 0u); });
    StaticFor<0, TM>::run([&](auto i) {
        read_a(i, Int<0>(), 0u);
        read_a(i, Int<1>(), 0u);
    });

    int sa = 0;                                                   // A slot of the current unit
    // One unit on B register set / B slot S.  Pairs of matrix instructions (the two K halves of one accumulator) are walked
    // row by row; the pairs after the first row carry the other instructions: DMA requests early, reads spread out.
    auto unit = [&](auto ss) {
        constexpr int S = decltype(ss)::value;
        auto& fa = f.a;
        auto& fb = f.b;
        asm volatile("s_waitcnt lgkmcnt(2)" ::: "memory");        // all but the last row of A
        hold_accumulators<TM * TN>();
        settle_b(ss);
#pragma unroll
        for (int i = 0; i + 1 < TM; ++i) asm volatile("" : "+v"(fa[0][i]), "+v"(fa[1][i]));
        const int sn = sa == 2 ? 0 : sa + 1;
        const uint32_t stage_a = sn * Cfg::A_BYTES, stage_b = (S ^ 1) * Cfg::B_BYTES;
        StaticFor<0, TM * TN>::run([&](auto pp) {
            constexpr int p = decltype(pp)::value, i = p / TN, jj = p % TN, j = (i & 1) ? TN - 1 - jj : jj;
            if constexpr (p == TN) {
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LA) : "memory");
                asm volatile("" : "+v"(fa[0][TM - 1]), "+v"(fa[1][TM - 1]));
                asm volatile("s_barrier" ::: "memory");
                hold_accumulators<TM * TN>();
            }
            mfma<i * TN + j>(fb[S][0][j], fa[0][i]);
            mfma<i * TN + j>(fb[S][1][j], fa[1][i]);
            if constexpr (p >= TN) {
                constexpr int q = p - TN, P = (TM - 1) * TN;
                if constexpr (jj == TN / 8) read_a(Int<i - 1>(), Int<0>(), stage_a);
                if constexpr (jj == TN / 8 + TN / 2) read_a(Int<i - 1>(), Int<1>(), stage_a);
                constexpr int PD = P * 4 / 7;                     // the pairs that carry DMA requests
                StaticFor<q * (LA + LB) / PD, (q + 1) * (LA + LB) / PD>::run([&](auto dd) {
                    constexpr int d = decltype(dd)::value;
                    if constexpr (d < LB) dma_b(S, d);
                    else if constexpr (d < LA + LB) dma_a(sa, d - LB);
                });
                StaticFor<q * Cfg::READS_B / P, (q + 1) * Cfg::READS_B / P>::run([&](auto r) { read_b(Int<S ^ 1>(), r, stage_b); });
            }
        });
        read_a(Int<TM - 1>(), Int<0>(), stage_a);
        read_a(Int<TM - 1>(), Int<1>(), stage_a);
        next_a();
        next_b();
        sa = sn;
    };
    for (int u = 0;;) {
        unit(Int<0>());
        if (++u == units) break;
        unit(Int<1>());
        if (++u == units) break;
    }
    // The last unit has read fragments of one that does not exist.  Nothing uses their registers, so they are free for the epilogue's
    // values from the read on, and a read that arrives late would overwrite those: nothing may be scheduled above the wait.  (The build
    // checks that no instruction touches them before it.  Used behind the wait as operands, so that they are not free, they take
    // the compiler's copies where the two ways out of the loop meet, in front of the wait, and spills.)
    // The last results need 18 wait states before a vector instruction reads them; the requests past the end have landed.
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    hold_accumulators<TM * TN>();
}

// ------------------------------------------------------------------------------------------------ epilogues
// Streaming (non-temporal) stores: what a large product writes does not fit the caches, and written through them it evicts
// the operands (8192^3, int32 out: 460 -> 395 us).
__device__ __forceinline__ void store4(int32_t* dst, const v4i& v) {
    __builtin_nontemporal_store(v, reinterpret_cast<v4i*>(dst));
}

// Whole lines.  A lane's four dwords x and y are 16 bytes of row l % 16 of two pieces of 64 bytes that lie next to each other
// in memory (two column tiles of fp32 or int32, two pairs of bf16 tiles).  Stored one after the other, every request writes 16
// half lines; instead the lanes of the rows r and r + 8 trade, so that `lower` is 8 rows (r) of whole 128-byte lines, and
// `upper` the other 8: lane l holds one of the four 16 bytes of piece (l / 8) % 2.
// 4096 x 4096 x 128, int32 out (67 MB, nothing but stores): 21.4 us with half lines, 16.9 with whole ones; 4096 x 14336 x 4096
// 229 and 214.  bf16 that stays in the caches: bf16_whole_lines.
template <class V>
__device__ __forceinline__ void whole_lines(const V& x, const V& y, V& lower, V& upper) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        lower[e] = __builtin_amdgcn_update_dpp((int)x[e], (int)y[e], 0x128, 0xF, 0xC, false);     // row_ror:8, lanes 8 .. 15
        upper[e] = __builtin_amdgcn_update_dpp((int)y[e], (int)x[e], 0x128, 0xF, 0x3, false);     // row_ror:8, lanes 0 .. 7
    }
}

// Plain epilogue: (float(acc) * row_scale[row]) * col_scale[col] -> fp32 or bf16, and / or the raw accumulators.
// PRE: the accumulator registers already hold the fp32 values to store, as bit patterns (lowrank_prepare).
// RAGGED: N is not a multiple of 16 (a tile's columns are then stored one by one); otherwise a 16-column tile lies inside
// the matrix or outside.  Its own instance, so that the code of the usual case stays short: every tile runs it once, from
// a cold instruction cache when there are few tiles.
template <class Cfg, bool PRE, bool RAGGED>
__device__ __forceinline__ void epilogue(const GemmArgs& a, const Place<Cfg>& at, int lane) {
    constexpr int TM = Cfg::TM, TN = Cfg::TN;
    // columns from the lane's first one of column tile j to the end of the matrix; without RAGGED the lane's position
    // inside the tile does not matter
    auto left_of = [&](int j) { return (int)(a.N - at.col(j)); };
    const int up = (lane >> 3) & 1;                               // the piece that the lane stores (whole_lines)
    const int64_t row_lo = at.row0 - 8 * up;                      // row of `lower`; that of `upper` is 8 further
    // one row of column tiles of 4-byte values
    auto store_row = [&](int32_t* base, int64_t ld, auto ii, const auto& value) {
        constexpr int i = decltype(ii)::value;
        __builtin_amdgcn_sched_barrier(0);                        // one row of tiles at a time
        hold_accumulators<TM * TN>();
        if constexpr (RAGGED) {
            if (at.row0 + 16 * i < a.M) {
                int32_t* row = base + (at.row0 + 16 * i) * ld;
                StaticFor<0, TN>::run([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    const v4i v = value(ii, jj);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e < left_of(j)) row[at.col(j) + e] = v[e];
                });
            }
        } else {
            const bool ok_lo = row_lo + 16 * i < a.M, ok_up = row_lo + 16 * i + 8 < a.M;
            int32_t* row = base + (row_lo + 16 * i) * ld + 16 * up;
            StaticFor<0, TN / 2>::run([&](auto hh) {
                constexpr int j = 2 * decltype(hh)::value;
                v4i lower, upper;
                whole_lines(value(ii, Int<j>()), value(ii, Int<j + 1>()), lower, upper);
                const bool in = left_of(j) > 16 * up;
                if (in && ok_lo) store4(row + at.col(j), lower);
                if (in && ok_up) store4(row + at.col(j) + 8 * ld, upper);
            });
        }
    };
    if constexpr (!PRE) {
        if (a.acc_out) {
            StaticFor<0, TM>::run([&](auto ii) {
                store_row(a.acc_out, a.ld_acc, ii, [](auto i, auto j) { return read_acc<decltype(i)::value * TN + decltype(j)::value>(); });
            });
        }
    }
    if (!a.C) return;
    v4f cs[TN];
    float rs[TM];
    if constexpr (!PRE) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            cs[j] = (v4f){1.0f, 1.0f, 1.0f, 1.0f};
            if (a.col_scale) {
                if constexpr (RAGGED) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e < left_of(j)) cs[j][e] = a.col_scale[at.col(j) + e];
                } else {
                    const float* p = a.col_scale + (left_of(j) > 0 ? at.col(j) : 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) cs[j][e] = p[e];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t row = at.row0 + 16 * i;
            rs[i] = a.row_scale ? a.row_scale[row < a.M ? row : a.M - 1] : 1.0f;
        }
    }
    auto values = [&](auto ii, auto jj) {
        constexpr int i = decltype(ii)::value, j = decltype(jj)::value;
        const v4i x = read_acc<i * TN + j>();
        v4f v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (PRE) v[r] = __int_as_float(x[r]);
            else v[r] = ((float)x[r] * rs[i]) * cs[j][r];
        }
        return v;
    };
    if (a.c_is_f32) {
        StaticFor<0, TM>::run([&](auto ii) {
            store_row(reinterpret_cast<int32_t*>(a.C), a.ldc, ii, [&](auto i, auto j) { return __builtin_bit_cast(v4i, values(i, j)); });
        });
        return;
    }
    // bf16: the four lanes of a row hold 4 x 4 columns of each tile, 8 bytes per lane.  Two column tiles at a time trade across
    // the lanes (one row-swap instruction per dword) so that a lane holds eight consecutive columns: lane groups 0 and 2 get
    // columns 0 .. 7 and 8 .. 15 of the first tile, groups 1 and 3 those of the second.
    const int shift = (lane >> 4) & 1 ? 12 : 0;                   // from the lane's first column of the first tile
    const int rows_left = (int)(a.M - row_lo < 65536 ? a.M - row_lo : 65536);
    auto pair_of = [&](auto ii, auto jj) {
        constexpr int j = decltype(jj)::value;
        const v4f x = values(ii, Int<j>()), y = values(ii, Int<j + 1>());
        v4u w;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const v2u t = __builtin_bit_cast(v2u, __builtin_amdgcn_permlane16_swap(pack_bf16x2(x[2 * h], x[2 * h + 1]),
                                                                                   pack_bf16x2(y[2 * h], y[2 * h + 1]), false, false));
            w[h] = t[0];
            w[2 + h] = t[1];
        }
        return w;
    };
    auto row_of_tiles = [&](auto ii, auto lines) {
        constexpr int i = decltype(ii)::value;
        __builtin_amdgcn_sched_barrier(0);                        // one row of tiles at a time
        hold_accumulators<TM * TN>();
        if constexpr (decltype(lines)::value == 0) {
            const bool row_ok = at.row0 + 16 * i < a.M;
            uint16_t* dst = reinterpret_cast<uint16_t*>(a.C) + (at.row0 + 16 * i) * a.ldc + shift;
            StaticFor<0, TN / 2>::run([&](auto hh) {
                constexpr int j = 2 * decltype(hh)::value;
                const v4u w = pair_of(ii, Int<j>());
                const int left = left_of(j) - shift;
                if constexpr (RAGGED) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (row_ok && e < left) dst[at.col(j) + e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                } else {
                    if (row_ok && left > 0) __builtin_nontemporal_store(w, reinterpret_cast<v4u*>(dst + at.col(j)));
                }
            });
        } else {
            const bool ok_lo = 16 * i < rows_left, ok_up = 16 * i + 8 < rows_left;
            uint16_t* dst = reinterpret_cast<uint16_t*>(a.C) + (row_lo + 16 * i) * a.ldc + shift + 32 * up;
            StaticFor<0, TN / 4>::run([&](auto hh) {
                constexpr int j = 4 * decltype(hh)::value;
                v4u lower, upper;
                whole_lines(pair_of(ii, Int<j>()), pair_of(ii, Int<j + 2>()), lower, upper);
                const bool in = left_of(j) - shift > 32 * up;
                if (in && ok_lo) __builtin_nontemporal_store(lower, reinterpret_cast<v4u*>(dst + at.col(j)));
                if (in && ok_up) __builtin_nontemporal_store(upper, reinterpret_cast<v4u*>(dst + at.col(j) + 8 * a.ldc));
            });
            if constexpr (TN % 4 != 0) {                          // two more, half a line that the other wavefront completes
                constexpr int j = TN - 2;
                const v4u w = pair_of(ii, Int<j>());
                uint16_t* half = reinterpret_cast<uint16_t*>(a.C) + (at.row0 + 16 * i) * a.ldc + shift + at.col(j);
                if (at.row0 + 16 * i < a.M && left_of(j) > shift) __builtin_nontemporal_store(w, reinterpret_cast<v4u*>(half));
            }
        }
    };
    if constexpr (!RAGGED) {
        if (a.whole_lines) {
            StaticFor<0, TM>::run([&](auto ii) { row_of_tiles(ii, Int<1>()); });
            return;
        }
    }
    StaticFor<0, TM>::run([&](auto ii) { row_of_tiles(ii, Int<0>()); });
}

// Eight values  x <- x + s * x[partner lane]  for the row stride 2^J inside groups of 16 lanes (row_of_lane), one rounded add or subtract each (the product with
// +-1 is exact).  A DPP read needs two wait states after a vector write of the same register: the leading s_nop supplies
// them for whatever came before; inside a block every register is used once.
template <int J>
__device__ __forceinline__ void lane_butterfly8(float& x0, float& x1, float& x2, float& x3, float& x4, float& x5, float& x6,
                                                float& x7, float s) {
#define HALO_DPP_FMAC8(CTRL)                                                                     \
    asm volatile("s_nop 1\n\t"                                                                   \
                 "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"              \
                 "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf"                   \
                 : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3), "+v"(x4), "+v"(x5), "+v"(x6), "+v"(x7) \
                 : "v"(s))
    if constexpr (J == 0) {
        HALO_DPP_FMAC8("quad_perm:[1,0,3,2]");
    } else if constexpr (J == 1) {
        HALO_DPP_FMAC8("quad_perm:[2,3,0,1]");
    } else if constexpr (J == 3) {
        HALO_DPP_FMAC8("row_ror:8");
    } else {
        HALO_DPP_FMAC8("row_half_mirror");                        // lane ^ 7: see row_of_lane
    }
#undef HALO_DPP_FMAC8
}

// Epilogue of a product whose output is then un-rotated on the left (level 2, E_X = H^T ( ... )): the accumulators are
// scaled, (float(acc) * row_scale[row]) * post_scale, and the eight lowest strides of the left-hand Walsh-Hadamard
// rotation run on the 256 rows of the tile before anything is stored, in ascending order and with every add and
// subtract a separately rounded fp32 operation, exactly as a pass over memory would do them.  Row index inside the
// tile = [wave_m | tile i (3 bits) | row in the tile (4 bits, lanes)], so strides 1 .. 8 pair lanes, 16, 32, 64 pair
// registers and 128 pairs this wavefront with the one holding the other 128 rows of the same columns, through LDS: each of
// the two hands over its second half of register tiles and finishes both rows' results of its first half (half the traffic
// of exchanging everything; the halves are in opposite order in the two, so both run the same code).
// Signs: a lane starts with its values multiplied by (-1)^(ones in its row number), folded into the row scale.  A pair's
// lanes then differ in sign, so the lower lane's own - partner is the wanted sum and the upper lane's own + partner the
// wanted difference, each up to the sign that the lower lane carries; after the fourth stage no sign is left.
// No normalisation: the 1/sqrt(block) of the rotation is applied after its last stride, by whoever runs it.
// N is a multiple of 16, M of 256.  SWAP placement.
template <class Cfg, bool PRE>
__device__ __forceinline__ void epilogue_left8(const GemmArgs& a, const Place<Cfg>& at, int wave, int lane,
                                               unsigned char* smem) {
    static_assert(Cfg::TM == 8 && Cfg::TN % 2 == 0, "256-row tiles");
    constexpr int TM = Cfg::TM, TN = Cfg::TN, HALF = TN / 2;
    static_assert(4 * TM * HALF * 1024 <= Cfg::LDS_BYTES, "exchange buffer");
    const int lrow = row_of_lane(lane & 15);
    const float sign = (__builtin_popcount(lrow) & 1) ? -1.0f : 1.0f;
    float rs[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) rs[i] = ((!PRE && a.row_scale) ? a.row_scale[at.row0 + 16 * i] : 1.0f) * sign;
    const bool scale_more = !PRE && a.post_scale;                 // uniform
    const float post = scale_more ? *a.post_scale : 1.0f;
    float s[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) s[b] = ((lrow >> b) & 1) ? 1.0f : -1.0f;

    // the stages inside the wavefront, on column tile j
    auto stages = [&](auto jj, float (&f)[TM][4]) {
        constexpr int j = decltype(jj)::value;
        __builtin_amdgcn_sched_barrier(0);                        // one column tile at a time
        hold_accumulators<TM * TN>();
        StaticFor<0, TM>::run([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            const v4i x = read_acc<i * TN + j>();
#pragma unroll
            for (int r = 0; r < 4; ++r) f[i][r] = (PRE ? __int_as_float(x[r]) : (float)x[r]) * rs[i];
        });
        if (scale_more) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) f[i][r] *= post;
        }
#pragma unroll
        for (int i = 0; i < TM; i += 2) {
            lane_butterfly8<0>(f[i][0], f[i][1], f[i][2], f[i][3], f[i + 1][0], f[i + 1][1], f[i + 1][2], f[i + 1][3], s[0]);
            lane_butterfly8<1>(f[i][0], f[i][1], f[i][2], f[i][3], f[i + 1][0], f[i + 1][1], f[i + 1][2], f[i + 1][3], s[1]);
            lane_butterfly8<2>(f[i][0], f[i][1], f[i][2], f[i][3], f[i + 1][0], f[i + 1][1], f[i + 1][2], f[i + 1][3], s[2]);
            lane_butterfly8<3>(f[i][0], f[i][1], f[i][2], f[i][3], f[i + 1][0], f[i + 1][1], f[i + 1][2], f[i + 1][3], s[3]);
        }
#pragma unroll
        for (int bit = 0; bit < 3; ++bit)
#pragma unroll
            for (int i = 0; i < TM; ++i)
                if ((i & (1 << bit)) == 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float x = f[i][r], y = f[i | (1 << bit)][r];
                        f[i][r] = x + y;
                        f[i | (1 << bit)][r] = x - y;
                    }
                }
    };
    v4f* xb = reinterpret_cast<v4f*>(smem);                       // [wavefront][j of the half][tile i][lane]
    __syncthreads();                                              // every wavefront is done with the operand stages
    StaticFor<0, HALF>::run([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        float f[TM][4];
        stages(Int<HALF + j>(), f);
#pragma unroll
        for (int i = 0; i < TM; ++i) xb[((wave * HALF + j) * TM + i) * 64 + lane] = (v4f){f[i][0], f[i][1], f[i][2], f[i][3]};
    });
    float kept[HALF][TM][4];
    StaticFor<0, HALF>::run([&](auto jj) { stages(jj, kept[decltype(jj)::value]); });
    __syncthreads();
    const v4f* other = xb + (wave ^ 2) * HALF * TM * 64 + lane;
    const float flip = wave >> 1 ? -1.0f : 1.0f;                  // the lower rows' wavefront: own - other; the upper's: other - own
    const int up = (lane >> 3) & 1;                               // whole lines, as in the plain epilogue
    int32_t* dst = reinterpret_cast<int32_t*>(a.C) + (at.row0 - 8 * up - (wave >> 1) * 128) * a.ldc + at.col_lo + 16 * up;
#pragma unroll
    for (int j = 0; j < HALF; j += 2) {
        __builtin_amdgcn_sched_barrier(0);
        if (at.col_lo + 16 * j < a.N) {
            const bool in = at.col_lo + 16 * (j + up) < a.N;
            int32_t* d = dst + 16 * j;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                v4i sum[2], dif[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const v4f o = other[((j + h) * TM + i) * 64];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        sum[h][r] = __float_as_int(kept[j + h][i][r] + o[r]);
                        dif[h][r] = __float_as_int((kept[j + h][i][r] - o[r]) * flip);
                    }
                }
                v4i sum_lo, sum_up, dif_lo, dif_up;
                whole_lines(sum[0], sum[1], sum_lo, sum_up);
                whole_lines(dif[0], dif[1], dif_lo, dif_up);
                if (in) {
                    store4(d, sum_lo);
                    store4(d + 8 * a.ldc, sum_up);
                    store4(d + 128 * a.ldc, dif_lo);
                    store4(d + 136 * a.ldc, dif_up);
                }
                d += 16 * a.ldc;
            }
        }
    }
}

// Low-rank side product (a LoRA branch next to the quantised product): turns the int32 accumulators, in place, into the
// fp32 values
//   ((float(acc) * row_scale[row]) * col_scale[col]) * post_scale  +  sum_k lr_a[row, k] * lr_b[k, col],
// the first part rounded exactly as the plain epilogues round it, the sum added by matrix instructions with the scaled
// accumulator as their addend.  The registers then hold float bit patterns and the PRE variants of the epilogues take
// over.
// The low-rank sum, 32 ranks at a time, by bf16 matrix instructions (v_mfma_f32_16x16x32_bf16: lane l supplies column /
// row l % 16, ranks 8 (l / 16) .. + 8; the result layout is that of the int8 instruction).  fp32 operands are split exactly
// into three bf16 pieces (8 + 8 + 8 mantissa bits, x = hi + mid + lo); every product of two pieces is exact and is
// accumulated in fp32.  The products kept are those down to 2^-16 of the full one (all of them when one operand is bf16
// already): what is dropped is below 2^-23 of |a b|, an fp32 rounding.  Smallest terms first.  Every address is clamped into
// its matrix, so that all loads are unconditional; what lies outside is zeroed afterwards.
// What bounds it: the latency of its loads, then its vector instructions.  All of them are requested before the first is used
// (the barriers keep the compiler from moving a load to its use) and land while the accumulators are scaled.
// The s_nop: two wait states between a vector write and a matrix instruction that reads it.
template <int T>
__device__ __forceinline__ void lowrank_mfma(const v8bf& bh, const v8bf& ah, const v8bf& am, const v8bf& al) {
    asm volatile("s_nop 1\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%4:%5], %0, %3, a[%4:%5]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%4:%5], %0, %2, a[%4:%5]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%4:%5], %0, %1, a[%4:%5]" ::"v"(bh), "v"(ah), "v"(am), "v"(al), "n"(4 * T),
                 "n"(4 * T + 3));
}
template <int T>
__device__ __forceinline__ void lowrank_mfma(const v8bf& bh, const v8bf& bm, const v8bf& bl, const v8bf& ah, const v8bf& am,
                                             const v8bf& al) {
    asm volatile("s_nop 1\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%6:%7], %0, %5, a[%6:%7]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%6:%7], %2, %3, a[%6:%7]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%6:%7], %1, %4, a[%6:%7]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%6:%7], %0, %4, a[%6:%7]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%6:%7], %1, %3, a[%6:%7]\n\t"
                 "v_mfma_f32_16x16x32_bf16 a[%6:%7], %0, %3, a[%6:%7]" ::"v"(bh), "v"(bm), "v"(bl), "v"(ah), "v"(am), "v"(al),
                 "n"(4 * T), "n"(4 * T + 3));
}
// B_BF16: lr_b is bf16 (the forward product, K-contiguous B) or fp32 (the E product, K-strided B).
template <class Cfg, bool B_BF16>
__device__ __forceinline__ void lowrank_prepare(const GemmArgs& a, const Place<Cfg>& at, int lane) {
    constexpr int TM = Cfg::TM, TN = Cfg::TN;
    const int l16 = lane & 15, g4 = lane >> 4;
    // ---- requests: scales and the first 32 ranks
    float rs[TM];
    v4f cs[TN], pa[TM][2];
    v4u pb[TN][B_BF16 ? 1 : 2];                                   // eight bf16 or fp32 values of lr_b
    auto request = [&](int c0) {
        const int kb = c0 + 8 * g4 < a.lr_rank ? c0 + 8 * g4 : 0; // the rank is a multiple of 8
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t row = at.row0 + 16 * i;
            const v4f* p = reinterpret_cast<const v4f*>(a.lr_a + (row < a.M ? row : a.M - 1) * a.lr_rank + kb);
            pa[i][0] = p[0];
            pa[i][1] = p[1];
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = at.col(j) - 4 * g4 + l16, at_b = (col < a.N ? col : a.N - 1) * a.lr_rank + kb;
            if constexpr (B_BF16) {
                pb[j][0] = *reinterpret_cast<const v4u*>(reinterpret_cast<const uint16_t*>(a.lr_b) + at_b);
            } else {
                const v4u* p = reinterpret_cast<const v4u*>(reinterpret_cast<const float*>(a.lr_b) + at_b);
                pb[j][0] = p[0];
                pb[j][1] = p[1];
            }
        }
    };
    const float post = a.post_scale ? *a.post_scale : 1.0f;                          // x * 1.0f is x
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int64_t row = at.row0 + 16 * i;
        rs[i] = a.row_scale ? a.row_scale[row < a.M ? row : a.M - 1] : 1.0f;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) cs[j] = (v4f){1.0f, 1.0f, 1.0f, 1.0f};
    if (a.col_scale) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const float* p = a.col_scale + (at.col(j) < a.N ? at.col(j) : 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) cs[j][e] = p[e];
        }
    }
    request(0);
    // ---- the scaled accumulators
    StaticFor<0, TN>::run([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        __builtin_amdgcn_sched_barrier(0);
        hold_accumulators<TM * TN>();
        StaticFor<0, TM>::run([&](auto ii) {
            constexpr int t = decltype(ii)::value * TN + j;
            v4i x = read_acc<t>();
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = __float_as_int((((float)x[r] * rs[decltype(ii)::value]) * cs[j][r]) * post);
            write_acc<t>(x);
        });
    });
    // ---- the low-rank sum
    auto hi16 = [](uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y, x, 0x07060302u); };
    auto split8 = [&](const v4f& x0, const v4f& x1, bool in, v8bf& h, v8bf& m, v8bf& l) {
        uint32_t ph[8], pm[8], pl[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float x = in ? (e < 4 ? x0[e & 3] : x1[e & 3]) : 0.0f;
            ph[e] = __float_as_uint(x) & 0xFFFF0000u;
            const float r1 = x - __uint_as_float(ph[e]);
            pm[e] = __float_as_uint(r1) & 0xFFFF0000u;
            pl[e] = __float_as_uint(r1 - __uint_as_float(pm[e]));
        }
        h = __builtin_bit_cast(v8bf, (v4u){hi16(ph[0], ph[1]), hi16(ph[2], ph[3]), hi16(ph[4], ph[5]), hi16(ph[6], ph[7])});
        m = __builtin_bit_cast(v8bf, (v4u){hi16(pm[0], pm[1]), hi16(pm[2], pm[3]), hi16(pm[4], pm[5]), hi16(pm[6], pm[7])});
        l = __builtin_bit_cast(v8bf, (v4u){hi16(pl[0], pl[1]), hi16(pl[2], pl[3]), hi16(pl[4], pl[5]), hi16(pl[6], pl[7])});
    };
    for (int c0 = 0;;) {
        const bool k_ok = c0 + 8 * g4 < a.lr_rank;
        v8bf ah[TM], am[TM], al[TM];
        __builtin_amdgcn_sched_barrier(0);
        hold_accumulators<TM * TN>();
#pragma unroll
        for (int i = 0; i < TM; ++i) split8(pa[i][0], pa[i][1], k_ok && at.row0 + 16 * i < a.M, ah[i], am[i], al[i]);
        StaticFor<0, TN>::run([&](auto jj) {
            constexpr int j = decltype(jj)::value;
            const bool in = k_ok && at.col(j) - 4 * g4 + l16 < a.N;
            if constexpr (B_BF16) {
                v4u raw = pb[j][0];
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[e] = in ? raw[e] : 0u;
                const v8bf bh = __builtin_bit_cast(v8bf, raw);
                StaticFor<0, TM>::run([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    lowrank_mfma<i * TN + j>(bh, ah[i], am[i], al[i]);
                });
            } else {
                v8bf bh, bm, bl;
                split8(__builtin_bit_cast(v4f, pb[j][0]), __builtin_bit_cast(v4f, pb[j][1]), in, bh, bm, bl);
                StaticFor<0, TM>::run([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    lowrank_mfma<i * TN + j>(bh, bm, bl, ah[i], am[i], al[i]);
                });
            }
        });
        hold_accumulators<TM * TN>();
        c0 += 32;
        if (c0 >= a.lr_rank) break;
        request(c0);
    }
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");             // as after the main loop
}

// ------------------------------------------------------------------------------------------------ kernel
template <class Cfg, bool TRANSB, bool LEFT, bool LR, bool RAGGED>
__device__ __forceinline__ void one_tile(const GemmArgs& a, int bid, int tiles_m, int tiles_n, unsigned char* smem) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int tile_m, tile_n;
    tile_of_block<Cfg::GROUP_M>(bid, tiles_m, tiles_n, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * Cfg::BM, n0 = (int64_t)tile_n * Cfg::BN;

    main_loop<Cfg, TRANSB, LEFT>(a, m0, n0, wave, lane, smem);
    const Place<Cfg> at(m0, n0, wave, lane, LEFT);
    if constexpr (LR) lowrank_prepare<Cfg, TRANSB>(a, at, lane);
    if constexpr (LEFT) {
        if (a.left_stages != 0) {          // uniform over the workgroup
            epilogue_left8<Cfg, LR>(a, at, wave, lane, smem);
            return;
        }
    }
    epilogue<Cfg, LR, RAGGED>(a, at, lane);
}

// LEFT: this instance also carries the epilogue that runs the low strides of a left-hand rotation.
// LR: this instance also carries the low-rank side product (lowrank_prepare).
// RAGGED: N (of either product) is not a multiple of 16.
// TN2: the second product of the launch has tiles of that width.
// The alignment: how fast these kernels run depends by up to 2 % on where in memory their instructions lie, whatever they are.  Steps of
// 2048 x 4096 x 4096, the pair of products, the same instructions: 63.8 us where the kernel began on a multiple of 32 KB, 65.2 and 65.6
// elsewhere; on another card 65.8 there, 67.1 in front of other kernels, and beginning on a multiple of 4 KB 66.7, 8 KB 65.9, 16 KB 66.9,
// 32 KB 67.0, 64 KB 66.3.
template <int TM, int TN, bool TRANSB, bool LEFT, bool LR, bool RAGGED, int TN2 = TN>
__global__ void __launch_bounds__(256, 1) __attribute__((aligned(8192)))
gemm_i8_kernel(GemmArgs a, int tiles_m, int tiles_n, GemmArgs a2, int tiles_m2, int tiles_n2, unsigned blocks1) {
    extern __shared__ __align__(16) unsigned char smem[];
    // A second, independent product may ride in the same launch (workgroups from blocks1 on): the tail and the
    // epilogue of one then overlap the main loop of the other.
    int bid = blockIdx.x;
    if (blockIdx.x >= blocks1) {
        bid -= blocks1;
        if constexpr (TN2 != TN) {
            one_tile<GemmCfg<TM, TN2, TRANSB>, TRANSB, LEFT, LR, RAGGED>(a2, bid, tiles_m2, tiles_n2, smem);
            return;
        }
        a = a2;
        tiles_m = tiles_m2;
        tiles_n = tiles_n2;
    }
    one_tile<GemmCfg<TM, TN, TRANSB>, TRANSB, LEFT, LR, RAGGED>(a, bid, tiles_m, tiles_n, smem);
}

// ------------------------------------------------------------------------------------------------ small products
// Products with too few 128 x 128 tiles to fill the chip: what bounds them is latency (of the first loads, of every unit of
// K, of the launch), not the matrix pipes.  A workgroup computes a 16 TM x 16 TN tile and its four wavefronts SPLIT K: wavefront
// w takes the units w, w + 4, ...  Each has an LDS ring of its own (two to eight stages of A and B, as many as LDS holds, filled
// and laid out as in the main kernel), so there is no barrier in the loop and all but one of the stages are in flight per wavefront
// from the start.  The four partial sums meet in LDS at the end, where every thread also picks up consecutive columns for the store.
// TM = 1 is for at most 16 rows (decode).  Tiles of 16 or 32 columns (TM up to 2, K-contiguous B): small_tile_columns.
template <int TM, int TN_, bool TRANSB>
struct SmallCfg {
    static constexpr int BM = 16 * TM, TN = TN_, BN = 16 * TN, BK = 128, SPLIT = 4;
    static constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, STAGE = A_BYTES + B_BYTES;
    static constexpr int LA = A_BYTES / 1024, LB = B_BYTES / 1024, L = LA + LB;  // DMA instructions per stage
    static constexpr int FIT = 150 / (SPLIT * L), NS = FIT > 8 ? 8 : FIT;        // ring stages: what LDS holds
    static constexpr int PITCH = BN + 4;                         // dwords per row of a partial sum
    static constexpr int RING_BYTES = SPLIT * NS * STAGE, SUM_BYTES = SPLIT * BM * PITCH * 4;
    static constexpr int LDS_BYTES = RING_BYTES > SUM_BYTES ? RING_BYTES : SUM_BYTES;
    static_assert(TRANSB || TN == 4, "rows of a K-strided B are fetched 64 columns at a time");
};

template <int TM, int TN_, bool TRANSB>
__global__ void __launch_bounds__(256)
gemm_i8_small_kernel(GemmArgs a, int tiles_n, GemmArgs a2, int tiles_n2, unsigned blocks1) {
    using Cfg = SmallCfg<TM, TN_, TRANSB>;
    constexpr int TN = Cfg::TN, BK = Cfg::BK, LA = Cfg::LA, LB = Cfg::LB, NS = Cfg::NS;
    unsigned bid = blockIdx.x;
    if (bid >= blocks1) {                  // the second product of a paired launch
        bid -= blocks1;
        a = a2;
        tiles_n = tiles_n2;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;
    const int64_t m0 = (int64_t)(bid / tiles_n) * Cfg::BM, n0 = (int64_t)(bid % tiles_n) * Cfg::BN;
    const uint32_t ring = (uint32_t)(uintptr_t)HALO_LDS_PTR(smem) + wave * NS * Cfg::STAGE;

    // ---- source offsets, as in main_loop, but every wavefront fetches the whole tile at its own K
    using KMajor = KMajorRequests<64>;                           // K-strided B: 16 rows of 64 bytes per request
    const int64_t rows_a = a.M - m0, rows_b = a.N - n0, cols_b = KMajor::columns(a.N, n0);
    const int r8 = lane >> 3, k0 = 16 * ((lane & 7) ^ (r8 >> 1));
    const int kc[2] = {k0, k0 ^ 64};
    const int krow = KMajor::first_row(0, lane, LB);
    uint32_t avo[LA], bvo[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i)
        avo[i] = r8 + 8 * i < rows_a ? (uint32_t)(r8 + 8 * i) * (uint32_t)a.lda + kc[i & 1] : kOutside;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        if constexpr (TRANSB) {
            bvo[i] = r8 + 8 * i < rows_b ? (uint32_t)(r8 + 8 * i) * (uint32_t)a.ldb + kc[i & 1] : kOutside;
        } else {
            bvo[i] = KMajor::offset(krow + 16 * i, KMajor::column(lane, i), a.ldb, cols_b);
        }
    }
    const int64_t b_unit = TRANSB ? (int64_t)BK : (int64_t)BK * a.ldb;
    const int units = (int)((a.K + Cfg::SPLIT * BK - 1) / (Cfg::SPLIT * BK));
    // 32-column tiles of a B whose rows lie a multiple of 8 KB apart: the tiles start at different K and go round, because at one
    // K all rows lie in the same few memory channels.  16 x 8192 x 8192, B in the caches 16.5 -> 12.5 us, from memory 17.5 -> 15.2;
    // 16 x 8192 x 16384 30.4 -> 22.1.  At other pitches, and with 16 columns, all tiles at one K are as fast or faster (16 x 4096 x
    // 8192 from memory 10.2 us, going round 13.3).
    constexpr bool ROUND = TRANSB && TN == 2;
    int first = 0;
    if constexpr (ROUND) {
        if (a.ldb % 8192 == 0 && a.K % (Cfg::SPLIT * BK) == 0) first = (int)(bid % tiles_n % (unsigned)units);
    }
    int to_end = units - first;
    v4u abuf = make_buffer(a.A + m0 * a.lda + wave * BK + first * (Cfg::SPLIT * BK));
    v4u bbuf = make_buffer((TRANSB ? a.B + n0 * a.ldb : a.B + n0) + wave * b_unit + first * (Cfg::SPLIT * BK));
    int64_t left = a.K - wave * BK;
    auto trim = [&]() {
        if (left >= BK) return;
#pragma unroll
        for (int i = 0; i < LA; ++i) avo[i] = kc[i & 1] < left ? avo[i] : kOutside;
#pragma unroll
        for (int i = 0; i < LB; ++i) bvo[i] = (TRANSB ? kc[i & 1] : krow + 16 * i) < left ? bvo[i] : kOutside;
    };
    auto request = [&](int slot) {
        trim();
        const uint32_t base = ring + slot * Cfg::STAGE;
#pragma unroll
        for (int i = 0; i < LB; ++i) dma16(bvo[i], bbuf, base + Cfg::A_BYTES + i * 1024);
#pragma unroll
        for (int i = 0; i < LA; ++i) dma16(avo[i], abuf, base + i * 1024);
        advance(abuf, Cfg::SPLIT * BK);
        advance(bbuf, Cfg::SPLIT * b_unit);
        left -= Cfg::SPLIT * BK;
        if constexpr (ROUND) {
            if (--to_end == 0 && first != 0) {
                advance(abuf, -a.K);
                advance(bbuf, -a.K);
            }
        }
    };
#pragma unroll
    for (int i = 0; i + 1 < NS; ++i) request(i);

    v4i acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = (v4i){0, 0, 0, 0};
    uint32_t a_addr[2], b_addr[TRANSB ? 2 : TN];
#pragma unroll
    for (int k = 0; k < 2; ++k) a_addr[k] = ring + l16 * BK + 16 * ((4 * k + g4) ^ (l16 >> 1));
    if constexpr (TRANSB) {
#pragma unroll
        for (int k = 0; k < 2; ++k) b_addr[k] = a_addr[k] + Cfg::A_BYTES;
    } else {
        const int row = 16 * g4 + (l16 >> 1);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            b_addr[j] = ring + Cfg::A_BYTES + row * Cfg::BN + 16 * (j ^ kmajor_swizzle<64>(row)) + 8 * (l16 & 1);
    }
    int slot = 0;
    for (int u = 0; u < units; ++u) {
        const int ahead = slot == 0 ? NS - 1 : slot - 1;         // (slot + NS - 1) % NS: read in the previous round
        request(ahead);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * Cfg::L) : "memory");
        const uint32_t st = slot * Cfg::STAGE;
        v4i fa[2][TM], fb[2][TN];
        v2i ft[2][TN][2];
        StaticFor<0, 2>::run([&](auto kk) {
            constexpr int k = decltype(kk)::value;
            auto& ra = fa;
            auto& rb = fb;
            auto& rt = ft;
            StaticFor<0, TM>::run([&](auto ii) {
                constexpr int i = decltype(ii)::value;
                lds_read16<i * 16 * BK>(ra[k][i], a_addr[k] + st);
            });
            StaticFor<0, TN>::run([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                if constexpr (TRANSB) {
                    lds_read16<j * 16 * BK>(rb[k][j], b_addr[k] + st);
                } else {
                    lds_read8_tr<k * 64 * Cfg::BN>(rt[k][j][0], b_addr[j] + st);
                    lds_read8_tr<k * 64 * Cfg::BN + 8 * Cfg::BN>(rt[k][j][1], b_addr[j] + st);
                }
            });
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(fa[k][i]));
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (TRANSB) {
                    asm volatile("" : "+v"(fb[k][j]));
                } else {
                    asm volatile("" : "+v"(ft[k][j][0]), "+v"(ft[k][j][1]));
                    fb[k][j] = (v4i){ft[k][j][0][0], ft[k][j][0][1], ft[k][j][1][0], ft[k][j][1][1]};
                }
            }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[k][j], fa[k][i], acc[i][j], 0, 0, 0);
        slot = slot == NS - 1 ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the requests past the end have landed
    __syncthreads();
    int32_t* sums = reinterpret_cast<int32_t*>(smem);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            *reinterpret_cast<v4i*>(sums + (wave * Cfg::BM + 16 * i + l16) * Cfg::PITCH + 16 * j + 4 * g4) = acc[i][j];
    __syncthreads();
    // ---- every thread: EPT consecutive columns of one row, VW at a time
    constexpr int EPT = TM * TN, TPR = Cfg::BN / EPT, VW = EPT < 4 ? EPT : 4, NV = EPT / VW;
    typedef int vi __attribute__((ext_vector_type(VW)));
    const int row_l = threadIdx.x / TPR, col_l = threadIdx.x % TPR * EPT;
    vi v[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
#pragma unroll
        for (int e = 0; e < VW; ++e) v[q][e] = 0;
#pragma unroll
        for (int w = 0; w < Cfg::SPLIT; ++w)
            v[q] += *reinterpret_cast<const vi*>(sums + (w * Cfg::BM + row_l) * Cfg::PITCH + col_l + VW * q);
    }
    const int64_t row = m0 + row_l, col = n0 + col_l;
    if (row >= a.M || col >= a.N) return;
    const bool whole = col + EPT <= a.N;
    auto store = [&](int32_t* dst, const vi(&x)[NV]) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            if (whole) {
                *reinterpret_cast<vi*>(dst + VW * q) = x[q];
            } else {
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    if (col + VW * q + e < a.N) dst[VW * q + e] = x[q][e];
            }
        }
    };
    if (a.acc_out) store(a.acc_out + row * a.ld_acc + col, v);
    if (!a.C) return;
    const float rs = a.row_scale ? a.row_scale[row] : 1.0f;
    vi f[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            const int64_t c = col + VW * q + e;
            const float cs = a.col_scale ? a.col_scale[c < a.N ? c : a.N - 1] : 1.0f;
            f[q][e] = __float_as_int(((float)v[q][e] * rs) * cs);
        }
    if (a.c_is_f32) {
        store(reinterpret_cast<int32_t*>(a.C) + row * a.ldc + col, f);
        return;
    }
    uint16_t* dst = reinterpret_cast<uint16_t*>(a.C) + row * a.ldc + col;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        uint32_t w[(VW + 1) / 2];
#pragma unroll
        for (int h = 0; h < VW / 2; ++h) w[h] = pack_bf16x2(__int_as_float(f[q][2 * h]), __int_as_float(f[q][2 * h + 1]));
        if constexpr (VW == 1) w[0] = bf16_bits(__int_as_float(f[q][0]));
        if (VW == 4 && whole) {
            *reinterpret_cast<v2u*>(dst + 4 * q) = (v2u){w[0], w[(VW - 1) / 2]};
        } else if (VW == 2 && whole) {
            *reinterpret_cast<uint32_t*>(dst + 2 * q) = w[0];
        } else {
#pragma unroll
            for (int e = 0; e < VW; ++e)
                if (col + VW * q + e < a.N) dst[VW * q + e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
        }
    }
}

// One thread per output, for what the tiles do not take: K = 0 (zeros), and row pitches so large that the rows of a tile do
// not fit one buffer's 4 GiB.
__global__ void __launch_bounds__(256) gemm_i8_plain_kernel(GemmArgs a) {
    const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (at >= a.M * a.N) return;
    const int64_t row = at / a.N, col = at % a.N;
    int acc = 0;
    for (int64_t k = 0; k < a.K; ++k)
        acc += (int)a.A[row * a.lda + k] * (int)(a.transB ? a.B[col * a.ldb + k] : a.B[k * a.ldb + col]);
    if (a.acc_out) a.acc_out[row * a.ld_acc + col] = acc;
    if (a.C) {
        const float v = ((float)acc * (a.row_scale ? a.row_scale[row] : 1.0f)) * (a.col_scale ? a.col_scale[col] : 1.0f);
        if (a.c_is_f32) reinterpret_cast<float*>(a.C)[row * a.ldc + col] = v;
        else reinterpret_cast<uint16_t*>(a.C)[row * a.ldc + col] = bf16_bits(v);
    }
}

// ------------------------------------------------------------------------------------------------ ceiling probe
// iters x 32 of the GEMM's matrix instructions per wavefront on operands read once from `operands` (4 KB: 16 bytes per lane
// and fragment, four fragments), nothing else in the loop: the rate the matrix pipes sustain on this machine for this
// operand data.
__global__ void __launch_bounds__(512) mfma_i8_probe_kernel(const int8_t* operands, int iters, int32_t* sink) {
    const int lane = threadIdx.x & 63;
    v4i f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const v4i*>(operands + (i * 64 + lane) * 16);
    v4i acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = (v4i){0, 0, 0, 0};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int m = 0; m < 32; ++m)
            acc[m / 2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[m % 2], f[2 + (m / 2) % 2], acc[m / 2], 0, 0, 0);
    }
    int s = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) s += acc[i][r];
    if (sink && s == 0x7fffffff) sink[0] = s;      // keeps the loop alive; practically never taken
}

// ------------------------------------------------------------------------------------------------ launch
// The dynamic-LDS limit of a kernel is raised once per kernel (and per process); call_once makes that safe when
// several host threads launch the same kernel for the first time.
template <class Kern>
hipError_t raise_lds_limit(Kern kern, int lds_bytes, std::once_flag* once, hipError_t* result) {
    std::call_once(*once, [&] {
        *result = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      lds_bytes);
    });
    return *result;
}

template <int TM, int TN, bool TRANSB, bool LEFT = false, bool LR = false, bool RAGGED = false>
hipError_t launch_tiles(const GemmArgs& a, hipStream_t s, const GemmArgs* a2 = nullptr) {
    using Cfg = GemmCfg<TM, TN, TRANSB>;
    const bool wants_left = a.left_stages != 0 || (a2 && a2->left_stages != 0);
    const bool wants_lr = a.lr_rank != 0 || (a2 && a2->lr_rank != 0);
    // the left-hand epilogue exists for K-strided B and 256 x 256 tiles
    constexpr bool kLeftShape = TM == 8 && TN == 8 && !TRANSB;
    if constexpr (!LR) {
        if (wants_lr) return launch_tiles<TM, TN, TRANSB, kLeftShape, true>(a, s, a2);
    }
    if constexpr (!LEFT && !LR && kLeftShape) {
        if (wants_left) return launch_tiles<TM, TN, TRANSB, true>(a, s, a2);
    }
    if (wants_left && !LEFT) return hipErrorInvalidValue;
    const bool ragged = a.N % 16 != 0 || (a2 && a2->N % 16 != 0);
    if constexpr (!LEFT && !LR && !RAGGED) {
        if (ragged) return launch_tiles<TM, TN, TRANSB, false, false, true>(a, s, a2);
    }
    if (ragged && !RAGGED) return hipErrorInvalidValue;
    auto lr_ok = [](const GemmArgs& g) {
        if (!LR) return true;
        return g.lr_rank > 0 && g.lr_rank <= kMaxLowRank && g.lr_rank % 8 == 0 && g.lr_a && g.lr_b &&
               (g.lr_b_bf16 != 0) == TRANSB && g.C && !g.acc_out;
    };
    if (!lr_ok(a) || (a2 && !lr_ok(*a2))) return hipErrorInvalidValue;
    static std::once_flag once;
    static hipError_t attr_result = hipSuccess;
    auto kern = gemm_i8_kernel<TM, TN, TRANSB, LEFT, LR, RAGGED>;
    hipError_t e = raise_lds_limit(kern, Cfg::LDS_BYTES, &once, &attr_result);
    if (e != hipSuccess) return e;
    // the epilogue that runs the low strides of a left-hand rotation: 256-row tiles that lie inside the matrix, fp32 out
    auto left_ok = [](const GemmArgs& g) {
        if (g.left_stages == 0) return true;
        return g.left_stages == 8 && g.M % 256 == 0 && g.C && g.c_is_f32 && !g.acc_out && (!g.col_scale || g.lr_rank) &&
               g.K > 0;
    };
    if (!left_ok(a) || (a2 && !left_ok(*a2))) return hipErrorInvalidValue;
    const int tiles_m = (int)((a.M + Cfg::BM - 1) / Cfg::BM), tiles_n = (int)((a.N + Cfg::BN - 1) / Cfg::BN);
    const unsigned blocks1 = (unsigned)(tiles_m * tiles_n);
    int tiles_m2 = 0, tiles_n2 = 0;
    if (a2) {
        tiles_m2 = (int)((a2->M + Cfg::BM - 1) / Cfg::BM);
        tiles_n2 = (int)((a2->N + Cfg::BN - 1) / Cfg::BN);
    }
    GemmArgs g = a, g2 = a2 ? *a2 : a;
    g.whole_lines = bf16_whole_lines(g.M, g.N, g.ldc);
    g2.whole_lines = bf16_whole_lines(g2.M, g2.N, g2.ldc);
    hipLaunchKernelGGL(kern, dim3(blocks1 + (unsigned)(tiles_m2 * tiles_n2)), dim3(Cfg::NT), Cfg::LDS_BYTES, s, g, tiles_m,
                       tiles_n, g2, tiles_m2, tiles_n2, blocks1);
    return hipGetLastError();
}

// The first `wide` columns in tiles of 256 x 256, the others in 256 x 192 (two_widths).
hipError_t launch_two_widths(const GemmArgs& a, int64_t wide, hipStream_t s) {
    if (a.left_stages != 0 || a.lr_rank != 0 || a.N % 16 != 0 || wide % 256 != 0 || wide >= a.N) return hipErrorInvalidValue;
    static std::once_flag once;
    static hipError_t attr_result = hipSuccess;
    constexpr int lds = GemmCfg<8, 8, true>::LDS_BYTES;
    auto kern = gemm_i8_kernel<8, 8, true, false, false, false, 6>;
    hipError_t e = raise_lds_limit(kern, lds, &once, &attr_result);
    if (e != hipSuccess) return e;
    GemmArgs g = a, g2 = a;
    g.whole_lines = bf16_whole_lines(a.M, a.N, a.ldc);
    g2.whole_lines = g.whole_lines;
    g.N = wide;
    g2.N -= wide;
    g2.B += wide * a.ldb;
    if (a.col_scale) g2.col_scale += wide;
    if (a.acc_out) g2.acc_out += wide;
    if (a.C) g2.C = static_cast<char*>(a.C) + wide * (a.c_is_f32 ? 4 : 2);
    const int tiles_m = (int)((a.M + 255) / 256), n1 = (int)(wide / 256), n2 = (int)((g2.N + 191) / 192);
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * (n1 + n2))), dim3(256), lds, s, g, tiles_m, n1, g2, tiles_m, n2,
                       (unsigned)(tiles_m * n1));
    return hipGetLastError();
}

template <int TM, bool TRANSB, int TN = 4>
hipError_t launch_small(const GemmArgs& a, hipStream_t s, const GemmArgs* a2 = nullptr) {
    using Cfg = SmallCfg<TM, TN, TRANSB>;
    if (a.left_stages != 0 || a.lr_rank != 0 || (a2 && (a2->left_stages != 0 || a2->lr_rank != 0))) return hipErrorInvalidValue;
    static std::once_flag once;
    static hipError_t attr_result = hipSuccess;
    auto kern = gemm_i8_small_kernel<TM, TN, TRANSB>;
    hipError_t e = raise_lds_limit(kern, Cfg::LDS_BYTES, &once, &attr_result);
    if (e != hipSuccess) return e;
    auto tiles = [](int64_t n, int t) { return (n + t - 1) / t; };
    const int64_t b1 = tiles(a.M, Cfg::BM) * tiles(a.N, Cfg::BN);
    const int64_t b2 = a2 ? tiles(a2->M, Cfg::BM) * tiles(a2->N, Cfg::BN) : 0;
    if (b1 + b2 > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)(b1 + b2)), dim3(256), Cfg::LDS_BYTES, s, a, (int)tiles(a.N, Cfg::BN), a2 ? *a2 : a,
                       (int)(a2 ? tiles(a2->N, Cfg::BN) : 1), (unsigned)b1);
    return hipGetLastError();
}

template <int TM, bool TRANSB>
hipError_t launch_small_by_columns(const GemmArgs& a, hipStream_t s) {
    if constexpr (TRANSB) {
        const int columns = small_tile_columns(a);
        if (columns == 16) return launch_small<TM, true, 1>(a, s);
        if (columns == 32) return launch_small<TM, true, 2>(a, s);
    }
    return launch_small<TM, TRANSB>(a, s);
}

inline bool tiles_can_run(const GemmArgs& a) {
    const int64_t most = ((int64_t(1) << 32) - 1024) / 256;       // 256 rows of a tile within one buffer
    return a.K > 0 && a.lda <= most && a.ldb <= most;
}

hipError_t launch_plain(const GemmArgs& a, hipStream_t s) {
    if (a.left_stages != 0 || a.lr_rank != 0) return hipErrorInvalidValue;
    const int64_t blocks = (a.M * a.N + 255) / 256;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_i8_plain_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

// K granularity of the tile configurations 0..3 that the ABI promises to refuse a K for (halo_gemm_config in halo.h).
constexpr int kStepOfConfig[4] = {64, 128, 128, 64};

template <bool TRANSB>
hipError_t launch_by_shape(const GemmArgs& a, hipStream_t s) {
    if constexpr (TRANSB) {
        const int64_t wide = two_widths(a);
        if (wide >= 0) return launch_two_widths(a, wide, s);
    }
    switch (a.config < 0 ? choose_config(a, nullptr) : a.config) {
        case 0:
        case 1: return launch_tiles<8, 8, TRANSB>(a, s);
        case 2: return launch_tiles<8, 4, TRANSB>(a, s);
        case 3:
        case 4: return launch_tiles<4, 4, TRANSB>(a, s);
        case kSmall64: return launch_small<4, TRANSB>(a, s);
        case kSmall32: return a.M <= 16 ? launch_small_by_columns<1, TRANSB>(a, s) : launch_small_by_columns<2, TRANSB>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool gemm_config_valid(int cfg, int64_t K) {
    if (cfg == -1 || cfg == 4) return true;
    return cfg >= 0 && cfg <= 3 && K % kStepOfConfig[cfg] == 0;
}

// Two K-strided-B products in one launch (the two backward products of the layer).  Falls back to two launches when
// the shapes do not allow the shared configuration.
hipError_t launch_gemm_i8_pair(const GemmArgs& a1, const GemmArgs& a2, hipStream_t s) {
    const bool ok = !a1.transB && !a2.transB && a1.M > 0 && a1.N > 0 && a2.M > 0 && a2.N > 0 && tiles_can_run(a1) && tiles_can_run(a2) &&
                    a1.config == a2.config && (a1.config == -1 || a1.config == 0 || a1.config == 3);
    if (!ok) {
        hipError_t e = launch_gemm_i8(a1, s);
        return e != hipSuccess ? e : launch_gemm_i8(a2, s);
    }
    switch (a1.config < 0 ? choose_config(a1, &a2) : a1.config) {
        case kSmall32: return launch_small<2, false>(a1, s, &a2);
        case kSmall64: return launch_small<4, false>(a1, s, &a2);
        case kTiles128: return launch_tiles<4, 4, false>(a1, s, &a2);
        default: return launch_tiles<8, 8, false>(a1, s, &a2);
    }
}

hipError_t launch_gemm_i8(const GemmArgs& a, hipStream_t s) {
    if (a.M == 0 || a.N == 0) return hipSuccess;
    if (!tiles_can_run(a)) return launch_plain(a, s);
    return a.transB ? launch_by_shape<true>(a, s) : launch_by_shape<false>(a, s);
}

hipError_t launch_mfma_i8_probe(const int8_t* operands, int iters, int32_t* sink, hipStream_t s) {
    hipLaunchKernelGGL(mfma_i8_probe_kernel, dim3(256), dim3(512), 0, s, operands, iters, sink);
    return hipGetLastError();
}

}  // namespace halo
