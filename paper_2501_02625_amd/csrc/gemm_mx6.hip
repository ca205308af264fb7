// MXFP6 GEMM on the CDNA4 scaled matrix instruction v_mfma_scale_f32_16x16x128_f8f6f4 with both operands in FP6 E3M2
// (format selector 3) and one E8M0 scale per block of 32 elements along K:  C = A B^T, fp32 accumulation.
//
// Operand layout of the instruction (established with a one-tile numeric probe against an exact reference): lane l
// supplies the 32 consecutive K-elements of row (l % 16) that start at K offset 32 * (l / 16), i.e. exactly one
// scaling block, as 192 bits packed least-significant element first in six registers, plus that block's E8M0 byte in
// byte 0 of the scale register.  Accumulator: lane l holds column (l % 16), rows 4 * (l / 16) + r, r = 0..3.
// So the packed codes in memory ([row][block][24 bytes]) are the register image: nothing is unpacked or shuffled.
// Three kernels: the one below for small products, and two of 256 x 256 tiles with DMA-fed LDS further down for large ones.
//
// Small products: workgroup = 4 wavefronts (2 x 2), macro tile 128 x 128, each wavefront 64 x 64 = 4 x 4 instruction tiles; K step 128
// elements = 96 code bytes + 4 scale bytes per row.  Two LDS stages: the 256 rows of a K step (128 of A, 128 of B) lie
// at a pitch of 112 bytes (28 dwords: the sixteen rows one quarter-wavefront reads fall on sixteen different groups of
// four banks), the scale dwords behind them.  The next K step travels global -> registers (six 16-byte loads and one
// scale dword per thread) while the current one is multiplied, then registers -> LDS, one barrier per K step.  A lane
// reads its block as three 8-byte LDS loads: the code bytes in memory are the register image, nothing is unpacked.
#include <mutex>

#include "halo_internal.h"
#include "matrix_asm.h"

namespace halo {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));

constexpr int kFmtE3M2 = 3;     // "bf6" in the instruction's format field (0 E4M3, 1 E5M2, 2 E2M3, 3 E3M2, 4 E2M1)
constexpr int kPitch = 112;                         // LDS bytes per row and K step
constexpr int kCodeBytes = 256 * kPitch;            // 128 rows of A, then 128 rows of B
constexpr int kStageBytes = kCodeBytes + 256 * 4;   // + one dword of four scale bytes per row

__global__ void __launch_bounds__(256, 2) gemm_mx6_kernel(Mx6GemmArgs a, int tiles_n) {
    __shared__ __align__(16) unsigned char smem[2 * kStageBytes];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const int r16 = lane & 15, g = lane >> 4;
    const int64_t m0 = (int64_t)(blockIdx.x / tiles_n) * 128;
    const int64_t n0 = (int64_t)(blockIdx.x % tiles_n) * 128;
    const int nk = (int)(a.K / 128);

    // ---- what this thread moves per K step: six 16-byte chunks of the 256 x 96 code bytes, one scale dword
    const uint8_t* src[6];
    int dst[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int q = tid + i * 256;                 // chunk number: row = q / 6, chunk of the row = q % 6
        const int row = q / 6, c = q % 6;
        int64_t gr;
        const uint8_t* base;
        int64_t ld;
        if (row < 128) { gr = m0 + row; gr = gr < a.M ? gr : a.M - 1; base = a.A; ld = a.lda; }
        else { gr = n0 + row - 128; gr = gr < a.N ? gr : a.N - 1; base = a.B; ld = a.ldb; }
        src[i] = base + gr * ld + c * 16;            // rows beyond the matrix are clamped; their results are never stored
        dst[i] = row * kPitch + c * 16;
    }
    const uint8_t* ssrc;
    {
        int64_t gr;
        if (tid < 128) { gr = m0 + tid; gr = gr < a.M ? gr : a.M - 1; ssrc = a.SA + gr * a.ldsa; }
        else { gr = n0 + tid - 128; gr = gr < a.N ? gr : a.N - 1; ssrc = a.SB + gr * a.ldsb; }
    }
    // two register sets: the loads of K step t+2 are in flight while step t is multiplied and step t+1 waits in the
    // other set for its turn to be written to LDS
    v4i reg0[6], reg1[6];
    uint32_t sreg0 = 0, sreg1 = 0;

    // ---- fragment addresses inside a stage (row tile t of A: rows wave_m*64 + 16t + r16; of B: 128 + wave_n*64 + ...)
    int fa_off[4], fb_off[4], sa_off[4], sb_off[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int ra = wave_m * 64 + t * 16 + r16, rb = 128 + wave_n * 64 + t * 16 + r16;
        fa_off[t] = ra * kPitch + g * 24; fb_off[t] = rb * kPitch + g * 24;
        sa_off[t] = kCodeBytes + ra * 4; sb_off[t] = kCodeBytes + rb * 4;
    }

    v4f acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    // One K step: request step kt+2 into `far` (free: its previous content went to LDS one step ago), multiply the
    // LDS stage of step kt, then hand step kt+1 (waiting in `near`) to the other LDS stage.
    // One K step (FAR = register set that receives step kt+2; the other one holds step kt+1): request step kt+2,
    // multiply the LDS stage of step kt, then hand step kt+1 to the other LDS stage.  Loads and LDS writes are
    // unconditional (beyond the last step they repeat the last one into a stage nobody reads any more).
#define HALO_MX6_K_STEP(KT, FAR, FAR_S, NEAR, NEAR_S)                                                                       \
    {                                                                                                                       \
        const int kt_ = (KT);                                                                                               \
        const int64_t koff = (int64_t)(kt_ + 2 < nk ? kt_ + 2 : nk - 1);                                                    \
        _Pragma("unroll") for (int i = 0; i < 6; ++i) FAR[i] = *reinterpret_cast<const v4i*>(src[i] + koff * 96);           \
        FAR_S = *reinterpret_cast<const uint32_t*>(ssrc + koff * 4);                                                        \
        const unsigned char* s = smem + (kt_ & 1) * kStageBytes;                                                            \
        v8i va[4], vb[4];                                                                                                   \
        int sa[4], sb[4];                                                                                                   \
        _Pragma("unroll") for (int t = 0; t < 4; ++t) {                                                                     \
            const uint2* pa = reinterpret_cast<const uint2*>(s + fa_off[t]);                                                \
            const uint2* pb = reinterpret_cast<const uint2*>(s + fb_off[t]);                                                \
            const uint2 a0 = pa[0], a1 = pa[1], a2 = pa[2], b0 = pb[0], b1 = pb[1], b2 = pb[2];                             \
            va[t] = v8i{(int)a0.x, (int)a0.y, (int)a1.x, (int)a1.y, (int)a2.x, (int)a2.y, 0, 0};                            \
            vb[t] = v8i{(int)b0.x, (int)b0.y, (int)b1.x, (int)b1.y, (int)b2.x, (int)b2.y, 0, 0};                            \
            sa[t] = (int)((*reinterpret_cast<const uint32_t*>(s + sa_off[t]) >> (8 * g)) & 0xFFu);                          \
            sb[t] = (int)((*reinterpret_cast<const uint32_t*>(s + sb_off[t]) >> (8 * g)) & 0xFFu);                          \
        }                                                                                                                   \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                                       \
            _Pragma("unroll") for (int j = 0; j < 4; ++j)                                                                   \
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(va[i], vb[j], acc[i][j], kFmtE3M2, kFmtE3M2,  \
                                                                             0, sa[i], 0, sb[j]);                           \
        __builtin_amdgcn_sched_barrier(0); /* the LDS writes (which wait for global data) stay behind the MFMAs */        \
        unsigned char* w = smem + ((kt_ + 1) & 1) * kStageBytes;                                                            \
        _Pragma("unroll") for (int i = 0; i < 6; ++i) *reinterpret_cast<v4i*>(w + dst[i]) = NEAR[i];                        \
        reinterpret_cast<uint32_t*>(w + kCodeBytes)[tid] = NEAR_S;                                                          \
        __syncthreads();                                                                                                    \
    }

    if (nk > 0) {
        const int64_t k1 = nk > 1 ? 1 : 0;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            reg0[i] = *reinterpret_cast<const v4i*>(src[i]);
            reg1[i] = *reinterpret_cast<const v4i*>(src[i] + k1 * 96);
        }
        sreg0 = *reinterpret_cast<const uint32_t*>(ssrc);
        sreg1 = *reinterpret_cast<const uint32_t*>(ssrc + k1 * 4);
#pragma unroll
        for (int i = 0; i < 6; ++i) *reinterpret_cast<v4i*>(smem + dst[i]) = reg0[i];
        reinterpret_cast<uint32_t*>(smem + kCodeBytes)[tid] = sreg0;
        __syncthreads();
        int kt = 0;
        for (; kt + 1 < nk; kt += 2) {
            HALO_MX6_K_STEP(kt, reg0, sreg0, reg1, sreg1)          // even step: step kt+1 waits in set 1, kt+2 goes to set 0
            HALO_MX6_K_STEP(kt + 1, reg1, sreg1, reg0, sreg0)
        }
        if (kt < nk) HALO_MX6_K_STEP(kt, reg0, sreg0, reg1, sreg1)
    }
#undef HALO_MX6_K_STEP

#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t col = n0 + wave_n * 64 + j * 16 + r16;
            if (col >= a.N) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t row = m0 + wave_m * 64 + i * 16 + 4 * g + r;
                if (row >= a.M) continue;
                if (a.c_is_f32) reinterpret_cast<float*>(a.C)[row * a.ldc + col] = acc[i][j][r];
                else reinterpret_cast<uint16_t*>(a.C)[row * a.ldc + col] = bf16_bits(acc[i][j][r]);
            }
        }
}


// ------------------------------------------------------------------------------------------------ large products
// 256 x 256 macro tile, 8 wavefronts (2 x 4), each 128 x 64 = 4 x 2 tiles of v_mfma_scale_f32_32x32x64_f8f6f4: twice
// the arithmetic per operand register of the 16x16x128 form.  Lane l of that instruction supplies the 32 consecutive
// K-elements (one scaling block, 24 bytes) of row l % 32 that start at K offset 32 * (l / 32); the accumulator has the
// usual 32 x 32 layout (lane l: column l % 32, rows 8 * (r / 4) + 4 * (l / 32) + r % 4 for r = 0..15).
//
// K step = 128 elements = 96 code bytes + 4 scale bytes per row.  Codes and scales travel global -> LDS by DMA
// (global_load_lds, 16 and 4 bytes per lane) through a ring of three stages, two K steps in flight.  A stage holds,
// per operand, 256 rows of 96 bytes, as they lie in memory: neighbouring lanes of a request fetch neighbouring 16-byte
// chunks of a row.  What bounds the kernel is the rate at which requests are turned into cache lines, and only lanes
// next to each other share one.  With planes of [16 rows][16 bytes] instead, where neighbouring lanes are 16 different
// rows, 8192 x 4096 x 4096 with both quantisers took 178.6 us; this way it takes 165.7.
// (Superblocks of 512 elements travel better: gemm_mx6_lines_kernel.)
// Rows r and r + 8 start on the same banks and rows 0..7 on eight different even groups of four, so rows with bit 3
// set have their chunks rotated by one place (big_place / big_chunk): a chunk of 16 rows then covers all 64 banks.  A
// lane reads its 24 bytes as three 8-byte pieces: the two halves of the wavefront (K blocks 2s and 2s+1 of sub-step s)
// always sit on complementary halves of the 16-byte chunks, so every such read covers all 64 banks evenly.
__device__ __forceinline__ int big_place(int chunk, int row) { return (chunk + ((row >> 3) & 1)) % 6; }
__device__ __forceinline__ int big_chunk(int place, int row) { return (place + 6 - ((row >> 3) & 1)) % 6; }
constexpr int kBigOpBytes = 256 * 96;                       // one operand's codes per stage
constexpr int kBigScaleOff = 2 * kBigOpBytes;               // 512 scale dwords (A rows, then B rows)
constexpr int kBigStage = kBigScaleOff + 512 * 4;
constexpr int kBigNS = 3;
constexpr int kBigLoads = 7;                                // DMA instructions per thread per K step
constexpr int kBigEpiPitch = 64 + 8;
constexpr int kBigLds = kBigNS * kBigStage;
static_assert(kBigLds <= 160 * 1024 && 8 * 32 * kBigEpiPitch * 4 <= kBigLds, "LDS budget");
#define HALO_GLOBAL_PTR(p) ((const __attribute__((address_space(1))) void*)(p))

typedef float v16f __attribute__((ext_vector_type(16)));

// The three 8-byte pieces of each of the six fragments (four of A, two of B) of one K sub-step.
struct BigFrags {
    v2i a[4][3], b[2][3];
};

// Requests the fragments of K sub-step KS (64 elements) of one stage.  addr_a / addr_b: LDS byte address of this
// lane's piece j of K block 2 * KS + half in the wavefront's first 32 rows; 32 rows are 3072 bytes apart.
// Issued as inline assembly: seen as LDS reads, the compiler would make them wait for every outstanding global->LDS
// transfer (s_waitcnt vmcnt(0)), which empties the ring at every K step.  big_wait_frags() waits for the data.
template <int KS>
__device__ __forceinline__ void big_load_frags(const uint32_t (&addr_a)[2][3], const uint32_t (&addr_b)[2][3], BigFrags& f) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
        asm volatile("ds_read_b64 %0, %4\n\tds_read_b64 %1, %4 offset:3072\n\t"
                     "ds_read_b64 %2, %4 offset:6144\n\tds_read_b64 %3, %4 offset:9216"
                     : "=&v"(f.a[0][j]), "=&v"(f.a[1][j]), "=&v"(f.a[2][j]), "=&v"(f.a[3][j])
                     : "v"(addr_a[KS][j]));
#pragma unroll
    for (int j = 0; j < 3; ++j)
        asm volatile("ds_read_b64 %0, %2\n\tds_read_b64 %1, %2 offset:3072"
                     : "=&v"(f.b[0][j]), "=&v"(f.b[1][j])
                     : "v"(addr_b[KS][j]));
}

// Waits for every outstanding LDS read.  The registers are operands of the wait, so nothing that uses them can move
// above it.
__device__ __forceinline__ void big_wait_frags(BigFrags& f) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(f.a[0][0]), "+v"(f.a[0][1]), "+v"(f.a[0][2]), "+v"(f.a[1][0]), "+v"(f.a[1][1]), "+v"(f.a[1][2]),
                   "+v"(f.a[2][0]), "+v"(f.a[2][1]), "+v"(f.a[2][2]), "+v"(f.a[3][0]), "+v"(f.a[3][1]), "+v"(f.a[3][2]),
                   "+v"(f.b[0][0]), "+v"(f.b[0][1]), "+v"(f.b[0][2]), "+v"(f.b[1][0]), "+v"(f.b[1][1]), "+v"(f.b[1][2]));
}

__device__ __forceinline__ v8i big_operand(const v2i (&p)[3]) {
    return v8i{p[0][0], p[0][1], p[1][0], p[1][1], p[2][0], p[2][1], 0, 0};
}

template <int KS>
__device__ __forceinline__ void big_mma(const BigFrags& f, const int (&sca)[4], const int (&scb)[2], v16f (&acc)[4][2]) {
    v8i va[4], vb[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) va[i] = big_operand(f.a[i]);
#pragma unroll
    for (int j = 0; j < 2; ++j) vb[j] = big_operand(f.b[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va[i], vb[j], acc[i][j], kFmtE3M2, kFmtE3M2,
                                                                        2 * KS, sca[i], 2 * KS, scb[j]);
}

__global__ void __launch_bounds__(512) gemm_mx6_big_kernel(Mx6GemmArgs a, int tiles_m, int tiles_n) {
    extern __shared__ __align__(16) unsigned char smem_big[];
    unsigned char* smem = smem_big;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wave_m = wave >> 2, wave_n = wave & 3;
    const int lrow = lane & 31, half = lane >> 5;

    int tile_m, tile_n;
    tile_of_block<4>(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * 256, n0 = (int64_t)tile_n * 256;
    const int nk = (int)(a.K / 128);

    // ---- per-thread DMA sources (fixed over the K loop): three 16-byte chunks of each operand, one scale dword.  Slot s
    // of an operand = row s / 6, place s % 6.  Rows beyond the matrix are clamped; their results are never stored.
    const uint8_t* a_src[3];
    const uint8_t* b_src[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int slot = tid + i * 512;
        const int row = slot / 6, c = big_chunk(slot % 6, row);
        int64_t gr = m0 + row;
        gr = gr < a.M ? gr : a.M - 1;
        a_src[i] = a.A + gr * a.lda + c * 16;
        gr = n0 + row;
        gr = gr < a.N ? gr : a.N - 1;
        b_src[i] = a.B + gr * a.ldb + c * 16;
    }
    const uint8_t* s_src;
    {
        int64_t gr;
        if (tid < 256) { gr = m0 + tid; gr = gr < a.M ? gr : a.M - 1; s_src = a.SA + gr * a.ldsa; }
        else { gr = n0 + tid - 256; gr = gr < a.N ? gr : a.N - 1; s_src = a.SB + gr * a.ldsb; }
    }
    // K step t (codes and scales of step `src`) into ring slot t % NS
    auto issue_dma = [&](int t, int src) {
        unsigned char* st = smem + (t % kBigNS) * kBigStage;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            __builtin_amdgcn_global_load_lds(HALO_GLOBAL_PTR(a_src[i] + (int64_t)src * 96),
                                             HALO_LDS_PTR(st + (wave * 64 + i * 512) * 16), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            __builtin_amdgcn_global_load_lds(HALO_GLOBAL_PTR(b_src[i] + (int64_t)src * 96),
                                             HALO_LDS_PTR(st + kBigOpBytes + (wave * 64 + i * 512) * 16), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(HALO_GLOBAL_PTR(s_src + (int64_t)src * 4),
                                         HALO_LDS_PTR(st + kBigScaleOff + wave * 64 * 4), 4, 0, 0);
    };

    // ---- this lane's three 8-byte pieces of K block 2 * ks + half, as byte offsets inside a stage
    uint32_t off_a[2][3], off_b[2][3], off_sa, off_sb;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int o = (2 * ks + half) * 24 + 8 * j;
            const uint32_t in_block = (uint32_t)(lrow * 96 + big_place(o / 16, lrow) * 16 + o % 16);
            off_a[ks][j] = (uint32_t)(wave_m * 4 * 3072) + in_block;
            off_b[ks][j] = (uint32_t)(kBigOpBytes + wave_n * 2 * 3072) + in_block;
        }
    off_sa = (uint32_t)(kBigScaleOff + (wave_m * 128 + lrow) * 4);
    off_sb = (uint32_t)(kBigScaleOff + (256 + wave_n * 64 + lrow) * 4);
    const uint32_t lds0 = (uint32_t)(uintptr_t)HALO_LDS_PTR(smem);

    v16f acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    if (nk > 0) {
        constexpr int D = kBigNS - 1;
        for (int t = 0; t < D; ++t) issue_dma(t, t < nk ? t : nk - 1);
        for (int kt = 0; kt < nk; ++kt) {
            // outstanding afterwards: the loads of step kt + 1 only
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((D - 1) * kBigLoads) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            // ring slot (kt - 1) % NS: everyone is past reading it
            issue_dma(kt + D, kt + D < nk ? kt + D : nk - 1);
            const uint32_t st = lds0 + (uint32_t)((kt % kBigNS) * kBigStage);
            uint32_t addr_a[2][3], addr_b[2][3];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int j = 0; j < 3; ++j) { addr_a[ks][j] = st + off_a[ks][j]; addr_b[ks][j] = st + off_b[ks][j]; }
            // the four scale bytes of each of this lane's six rows (same inline-assembly reasoning as the fragments)
            int sca[4], scb[2];
            asm volatile("ds_read_b32 %0, %6\n\tds_read_b32 %1, %6 offset:128\n\tds_read_b32 %2, %6 offset:256\n\t"
                         "ds_read_b32 %3, %6 offset:384\n\tds_read_b32 %4, %7\n\tds_read_b32 %5, %7 offset:128"
                         : "=&v"(sca[0]), "=&v"(sca[1]), "=&v"(sca[2]), "=&v"(sca[3]), "=&v"(scb[0]), "=&v"(scb[1])
                         : "v"(st + off_sa), "v"(st + off_sb));
            BigFrags f0, f1;
            big_load_frags<0>(addr_a, addr_b, f0);
            big_wait_frags(f0);              // the hardware counts at most 15 outstanding LDS reads: no partial wait here
            asm volatile("" : "+v"(sca[0]), "+v"(sca[1]), "+v"(sca[2]), "+v"(sca[3]), "+v"(scb[0]), "+v"(scb[1]));
            big_load_frags<1>(addr_a, addr_b, f1);       // in flight while sub-step 0 is multiplied
#pragma unroll
            for (int i = 0; i < 4; ++i) sca[i] = (int)((uint32_t)sca[i] >> (8 * half));
#pragma unroll
            for (int j = 0; j < 2; ++j) scb[j] = (int)((uint32_t)scb[j] >> (8 * half));
            big_mma<0>(f0, sca, scb, acc);
            big_wait_frags(f1);
            big_mma<1>(f1, sca, scb, acc);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    }

    // ---- epilogue: each wavefront drops a 32-row slab of its sub-tile into a private LDS region and reads it back four
    // consecutive columns per lane, so the global stores are 16-byte (fp32) or 8-byte (bf16) pieces of covered rows
    __syncthreads();
    float* region = reinterpret_cast<float*>(smem) + wave * 32 * kBigEpiPitch;
    const int cc = (lane % 16) * 4;
    const int64_t col = n0 + wave_n * 64 + cc;
    const bool col_any = col < a.N, col_all = col + 4 <= a.N;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) region[(8 * (r / 4) + 4 * half + (r % 4)) * kBigEpiPitch + j * 32 + lrow] = acc[i][j][r];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int rr = p * 4 + lane / 16;
            const float4 v = *reinterpret_cast<const float4*>(region + rr * kBigEpiPitch + cc);
            const int64_t row = m0 + wave_m * 128 + i * 32 + rr;
            if (row >= a.M || !col_any) continue;
            const float f[4] = {v.x, v.y, v.z, v.w};
            if (a.c_is_f32) {
                float* dst = reinterpret_cast<float*>(a.C) + row * a.ldc + col;
                if (col_all) {
                    *reinterpret_cast<float4*>(dst) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < a.N) dst[e] = f[e];
                }
            } else {
                uint16_t* dst = reinterpret_cast<uint16_t*>(a.C) + row * a.ldc + col;
                if (col_all) {
                    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(f[0], f[1]),
                                                                 pack_bf16x2(f[2], f[3]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < a.N) dst[e] = bf16_bits(f[e]);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------ large products, whole lines
// K a multiple of 512.  256 x 256 macro tile, four wavefronts (2 x 2) of 128 x 128 = 4 x 4 tiles of 32 x 32, one per SIMD, the
// 256 accumulators in named accumulation registers as in the INT8 kernel.
//
// What travels is not a K step (96 bytes of a row, which touch 1.5 cache lines on average, and every line is fetched again for
// the next step) but a LINE: 128 bytes of each of the 512 rows.  Nothing but the transfers of 8192 x 4096 x 4096 takes 63 us in
// pieces of 96 bytes with two K steps on their way, 48 in lines with one line on its way.
// A SUPERBLOCK is three lines = 512 elements = 16 scaling blocks = eight GROUPS of 64 elements (one matrix instruction deep).  The
// bytes of group g are 48 g .. 48 g + 47 of the superblock: groups 0, 1 lie in line 0; 3, 4 in line 1; 6, 7 in line 2; 2 and 5
// across two of them.  LDS holds two lines of both operands, line n of the product in slot n % 2.  A slot is wanted again for the
// line after next, so what a straddling group has in the older line is read ahead: group 2 is read whole from line 0, with garbage
// where line 1 has not come, and the two pieces of its upper half-wavefront that lie in line 1 are read again under an execution
// mask; group 5 likewise.  Fragments live in three register sets, group g in set kLineSet[g].
// By the group that is being multiplied (16 matrix instructions), what is read meanwhile, and at which barrier a line is requested:
//   0: group 1
//   1: [line 1 has landed and line 0's slot is free: line 2 is requested] the rest of 2, 3
//   2: 3, 4
//   3: 4, 5 as far as line 1 goes
//   4: [line 2 has landed, line 1's slot is free: line 0 and the scales of the next superblock] the rest of 5, 6
//   5: 6, 7
//   6: [that line 0 has landed, line 2's slot is free: line 1 of the next superblock] the next group 2
//   7: the next group 0
// Three barriers a superblock, each behind a wait for everything requested: one line (64 KB) is always on its way.  As in the INT8
// kernel everything is inline assembly in program order.
//
// What bounds it: power.  The matrix instructions alone, operands in registers, sustain 5.3 PFLOP/s on random codes (9.2 on zeros),
// and the parts add up rather than overlap: 8192 x 4096 x 4096, bf16 out, 90 us; without the transfers 78, without the LDS reads 76,
// matrix instructions only 55, transfers only 69, reads only 53; barriers and requests earlier, later or denser change nothing.  The
// eight-wavefront kernel above takes 118.
//
// LDS: row r of a line at 128 r, its 16-byte chunk c at place (c + r / 2) % 8.  A lane's 24 bytes of a group are three 8-byte pieces;
// the two halves of a wavefront always sit on complementary halves of the chunks, and sixteen rows on sixteen different groups of
// banks.  B is passed as the instruction's first operand: a lane holds row l % 32 of C, columns 8 q + 4 (l / 32) .. + 3.
constexpr int kLineSlot = 256 * 128;                        // one operand's line
constexpr int kLineScales = 4 * kLineSlot;                  // two buffers of 512 rows x 16 scale bytes (one superblock)
constexpr int kLinesLds = kLineScales + 2 * 512 * 16;
constexpr int kLineEpiPitch = 128 + 4;                      // dwords
static_assert(kLinesLds <= 160 * 1024 && 4 * 32 * kLineEpiPitch * 4 <= kLinesLds, "LDS budget");
constexpr int kLineSet[8] = {0, 1, 2, 0, 1, 2, 0, 1};

typedef int v6i __attribute__((ext_vector_type(6)));

struct LineFrags {
    v2i a[4][3], b[4][3];
};

// What a wavefront reads while it multiplies a group: a list of fragment pieces.  Fragment f: 0 .. 3 of B, 4 .. 7 of A.
enum LineRead { kScale, kWhole, kHigh12, kLow01, kPiece2, kHigh01 };
struct LineOp {
    int kind, group, f;
};
struct LineOps {
    int n;
    LineOp op[40];
};
// The reads of slot g in order.  kWhole: three pieces of a fragment (24 bytes of a lane); kHigh12, kHigh01: two pieces, upper half-wavefront
// only; kLow01: two pieces; kPiece2: one.
constexpr LineOps line_ops(int g) {
    LineOps r{};
    auto add = [&r](int kind, int group, int from, int to) {
        for (int f = from; f < to; ++f) r.op[r.n++] = LineOp{kind, group, f};
    };
    if (g & 1) add(kScale, (g + 1) & 7, 0, 8);
    switch (g) {
        case 0: add(kWhole, 1, 0, 8); break;
        case 1: add(kHigh12, 2, 0, 8); add(kWhole, 3, 0, 3); break;
        case 2: add(kWhole, 3, 3, 8); add(kWhole, 4, 0, 5); break;
        case 3: add(kWhole, 4, 5, 8); add(kLow01, 5, 0, 8); break;
        case 4: add(kPiece2, 5, 0, 8); add(kHigh01, 5, 0, 8); add(kWhole, 6, 0, 4); break;
        case 5: add(kWhole, 6, 4, 8); add(kWhole, 7, 0, 8); break;
        case 6: add(kWhole, 2, 0, 8); break;
        default: add(kWhole, 0, 0, 8); break;
    }
    return r;
}
constexpr int line_reads(int kind) { return kind == kWhole ? 3 : kind == kScale || kind == kPiece2 ? 1 : 2; }
// LDS reads that are requested after the last one of group g until slot g begins: what a wait for that group may leave
// outstanding (the counter holds 15).
constexpr int line_reads_after(int g) {
    int n = 0;
    for (int s = g + 7;; --s) {
        const LineOps o = line_ops(s & 7);
        for (int q = o.n - 1; q >= 0; --q) {
            if (o.op[q].kind != kScale && o.op[q].group == g) return n < 15 ? n : 15;
            n += line_reads(o.op[q].kind);
        }
    }
}
// What slot g requests after its matrix instructions 0 .. m - 1 have been issued, `first` being the first that is followed by reads.
constexpr int line_ops_before(int g, int first, int m) { return m <= first ? 0 : (m - first) * line_ops(g).n / (14 - first); }
constexpr int line_reads_before(int g, int first, int m) {
    const LineOps o = line_ops(g);
    int n = 0;
    for (int q = 0; q < line_ops_before(g, first, m); ++q) n += line_reads(o.op[q].kind);
    return n < 15 ? n : 15;
}
template <int G>
struct LineSlot {
    static constexpr LineOps OPS = line_ops(G);
};

template <int T, int HI>
__device__ __forceinline__ void line_mfma(const v6i& b, const v6i& a, int sb, int sa) {
    if constexpr (HI)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 a[%4:%5], %0, %1, a[%4:%5], %2, %3 op_sel_hi:[1,1,0] cbsz:3 blgp:3" ::"v"(b),
                     "v"(a), "v"(sb), "v"(sa), "n"(16 * T), "n"(16 * T + 15));
    else
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 a[%4:%5], %0, %1, a[%4:%5], %2, %3 op_sel_hi:[0,0,0] cbsz:3 blgp:3" ::"v"(b),
                     "v"(a), "v"(sb), "v"(sa), "n"(16 * T), "n"(16 * T + 15));
}
template <int OFF>
__device__ __forceinline__ void line_read(v2i& d, uint32_t addr) {
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
// Two reads for lanes 32 .. 63 only.
template <int OFF>
__device__ __forceinline__ void line_read_high(v2i& d0, v2i& d1, uint32_t addr0, uint32_t addr1) {
    asm volatile("s_mov_b32 exec_lo, 0\n\tds_read_b64 %0, %2 offset:%4\n\tds_read_b64 %1, %3 offset:%4\n\ts_mov_b32 exec_lo, -1"
                 : "+v"(d0), "+v"(d1)
                 : "v"(addr0), "v"(addr1), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void line_read_scale(int& d, uint32_t addr) {
    asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}

__global__ void __launch_bounds__(256, 1) gemm_mx6_lines_kernel(Mx6GemmArgs a, int tiles_m, int tiles_n) {
    extern __shared__ __align__(128) unsigned char smem_big[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const int lrow = lane & 31, half = lane >> 5;
    int tile_m, tile_n;
    tile_of_block<4>(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * 256, n0 = (int64_t)tile_n * 256;
    const uint32_t lds = (uint32_t)(uintptr_t)HALO_LDS_PTR(smem_big);

    // ---- requests: eight of 8 rows x 128 bytes per operand and line, two of 64 rows x 16 scale bytes per superblock.  Rows beyond
    // the matrix come as zeros, and so does everything once the last line has been requested.
    uint32_t avo[8], bvo[8], svo[2];
    {
        const int r8 = lane >> 3, k0 = 16 * (((lane & 7) - (r8 >> 1)) & 7), row = wave * 64 + r8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t k = (uint32_t)(k0 ^ ((i & 1) << 6)), r = (uint32_t)(row + 8 * i);
            avo[i] = m0 + r < a.M ? r * (uint32_t)a.lda + k : kOutside;
            bvo[i] = n0 + r < a.N ? r * (uint32_t)a.ldb + k : kOutside;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = (wave & 1) * 128 + 64 * i + lane;
            svo[i] = wave < 2 ? (m0 + r < a.M ? (uint32_t)r * (uint32_t)a.ldsa : kOutside)
                              : (n0 + r < a.N ? (uint32_t)r * (uint32_t)a.ldsb : kOutside);
        }
    }
    v4u abuf = make_buffer(a.A + m0 * a.lda), bbuf = make_buffer(a.B + n0 * a.ldb);
    v4u sbuf = make_buffer(wave < 2 ? a.SA + m0 * a.ldsa : a.SB + n0 * a.ldsb);
    int supers = (int)(a.K / 512), lines = 3 * supers, scales = supers;      // still to do / to be requested
    auto request = [&](auto slot, auto dd) {                     // request dd of a line into a slot
        constexpr int d = decltype(dd)::value, i = d & 7, at = (decltype(slot)::value + (d >> 3) * 2) * kLineSlot + i * 1024;
        if constexpr (d < 8) dma16(avo[i], abuf, lds + at + wave * 8192);
        else dma16(bvo[i], bbuf, lds + at + wave * 8192);
    };
    auto next_line = [&]() {
        advance(abuf, 128);
        advance(bbuf, 128);
        if (--lines == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) avo[i] = bvo[i] = kOutside;
        }
    };
    auto request_scales = [&](auto buffer) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            dma16(svo[i], sbuf, lds + kLineScales + decltype(buffer)::value * 8192 + wave * 2048 + i * 1024);
        advance(sbuf, 16);
        if (--scales == 0) svo[0] = svo[1] = kOutside;
    };
    request_scales(Int<0>());
    StaticFor<0, 16>::run([&](auto d) { request(Int<0>(), d); });
    next_line();
    StaticFor<0, 16>::run([&](auto d) { request(Int<1>(), d); });
    next_line();
    hold_accumulators<64>();
    StaticFor<0, 64>::run([&](auto t) { clear_acc<decltype(t)::value>(); });

    // ---- where a lane's pieces lie: piece j of group g in chunk 3 g + d, d and the half of the chunk fixed by j and the half-wavefront
    uint32_t piece[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int byte = 24 * half + 8 * j;
        piece[j] = (uint32_t)(16 * (byte / 16 + ((lrow >> 1) & 7)) + byte % 16);
    }
    const uint32_t rows_a = lds + (uint32_t)(wave_m * 128 + lrow) * 128;
    const uint32_t rows_b = lds + 2 * kLineSlot + (uint32_t)(wave_n * 128 + lrow) * 128;
    const uint32_t scale_a = lds + kLineScales + (uint32_t)(wave_m * 128 + lrow) * 16;
    const uint32_t scale_b = lds + kLineScales + (uint32_t)(256 + wave_n * 128 + lrow) * 16;
    const int shift = 8 * half;
    LineFrags f[3];
    int sc[2][8];                                                // scale bytes of a pair of groups: B's four rows, A's four
    struct Addr {
        uint32_t a[3], b[3];
    };
    auto address = [&](auto gg, Addr& at) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            asm volatile("" : "+v"(piece[j]));                   // not hoisted out of the loop: 48 registers
            const uint32_t in_row = (piece[j] + 48u * decltype(gg)::value) & 127u;
            at.a[j] = in_row | rows_a;
            at.b[j] = in_row | rows_b;
        }
    };
    // one entry of line_ops(G); P: parity of the superblock
    auto read = [&](auto gg, auto pp, auto qq, const Addr& at) {
        constexpr int G = decltype(gg)::value, P = decltype(pp)::value;
        constexpr LineOp op = LineSlot<G>::OPS.op[decltype(qq)::value];
        constexpr int fr = op.f & 3, set = kLineSet[op.group];
        if constexpr (op.kind == kScale) {
            constexpr int off = (op.group == 0 ? 1 - P : P) * 8192 + fr * 512 + (op.group / 2) * 4;
            line_read_scale<off>(sc[(op.group / 2) & 1][op.f], op.f < 4 ? scale_b : scale_a);
        } else {
            // the line the pieces come from: of this superblock 0, 1, 2 in slots P, 1 - P, P; the next one's line 0 in 1 - P
            constexpr int slot = G == 0 || (G >= 4 && G <= 5) ? P : 1 - P;
            constexpr int off = slot * kLineSlot + fr * 4096;
            auto& ad = op.f < 4 ? at.b : at.a;
            auto& d = op.f < 4 ? f[set].b[fr] : f[set].a[fr];
            if constexpr (op.kind == kWhole || op.kind == kLow01) {
                line_read<off>(d[0], ad[0]);
                line_read<off>(d[1], ad[1]);
            }
            if constexpr (op.kind == kWhole || op.kind == kPiece2) line_read<off>(d[2], ad[2]);
            if constexpr (op.kind == kHigh12) line_read_high<off>(d[1], d[2], ad[1], ad[2]);
            if constexpr (op.kind == kHigh01) line_read_high<off>(d[0], d[1], ad[0], ad[1]);
        }
    };
    // Fragments [from, to) of a set: valid from here on, and each in six registers in a row.  The nop: whatever the compiler copies to
    // bring that about stands before it, and a vector write needs two wait states before a matrix instruction reads it.
    auto settle = [&](auto ss, auto from, auto to, v6i (&t)[8]) {
        auto& fs = f[decltype(ss)::value];
#pragma unroll
        for (int i = decltype(from)::value; i < decltype(to)::value; ++i) {
            v2i(&p)[3] = i < 4 ? fs.b[i & 3] : fs.a[i & 3];
#pragma unroll
            for (int j = 0; j < 3; ++j) asm volatile("" : "+v"(p[j]));
            t[i] = (v6i){p[0][0], p[0][1], p[1][0], p[1][1], p[2][0], p[2][1]};
            asm volatile("" : "+v"(t[i]));
        }
        asm volatile("s_nop 1" ::: "memory");
    };

    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");            // line 0 and the scales
    asm volatile("s_barrier" ::: "memory");
    {
        Addr at;
        StaticFor<0, 8>::run([&](auto q) { read(Int<7>(), Int<1>(), q, at); });          // the scales of groups 0 and 1
        address(Int<2>(), at);
        StaticFor<0, LineSlot<6>::OPS.n>::run([&](auto q) { read(Int<6>(), Int<1>(), q, at); });
        address(Int<0>(), at);
        StaticFor<8, LineSlot<7>::OPS.n>::run([&](auto q) { read(Int<7>(), Int<1>(), q, at); });
    }

    // One group: 16 matrix instructions, row by row of A's fragments, the other instructions between them.
    auto group = [&](auto gg, auto pp) {
        constexpr int G = decltype(gg)::value, P = decltype(pp)::value, SET = kLineSet[G];
        constexpr LineOps ops = LineSlot<G>::OPS;
        // the first group whose pieces are read here, and the second
        constexpr int G1 = ops.op[(G & 1) ? 8 : 0].group, G2 = ops.op[ops.n - 1].group;
        constexpr int barrier = (G == 1 || G == 4) ? 4 : G == 6 ? 6 : -1;      // before this matrix instruction
        constexpr int slot = G == 4 ? 1 - P : P;                 // of the line requested behind the barrier
        constexpr int first = barrier < 0 ? 0 : barrier;         // matrix instruction behind which the reads begin
        // groups 0 and 1 were read last: all but the last two fragments of A
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(G <= 1 ? 6 : line_reads_after(G)) : "memory");
        hold_accumulators<64>();
        if constexpr ((G & 1) == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                asm volatile("v_lshrrev_b32 %0, %1, %0" : "+v"(sc[(G / 2) & 1][i]) : "v"(shift));
            }
        }
        Addr at1, at2;
        address(Int<G1>(), at1);
        if constexpr (G2 != G1) address(Int<G2>(), at2);
        v6i t[8];
        settle(Int<SET>(), Int<0>(), Int<(G <= 1 ? 6 : 8)>(), t);
        StaticFor<0, 16>::run([&](auto mm) {
            constexpr int m = decltype(mm)::value, i = m >> 2, j = (i & 1) ? 3 - (m & 3) : m & 3;
            if constexpr (m == barrier) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                asm volatile("s_barrier" ::: "memory");
                hold_accumulators<64>();
            }
            if constexpr (G <= 1 && m == 8) {
                asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(line_reads_before(G, first, m)) : "memory");
                settle(Int<SET>(), Int<6>(), Int<8>(), t);
            }
            line_mfma<4 * i + j, G & 1>(t[j], t[4 + i], sc[(G / 2) & 1][j], sc[(G / 2) & 1][4 + i]);
            if constexpr (m >= first && m < 14) {
                StaticFor<line_ops_before(G, first, m), line_ops_before(G, first, m + 1)>::run([&](auto q) {
                    constexpr LineOp op = LineSlot<G>::OPS.op[decltype(q)::value];
                    if constexpr (op.group == G1 || op.kind == kScale) read(gg, pp, q, at1);
                    else read(gg, pp, q, at2);
                });
            }
            if constexpr (barrier >= 0 && m >= barrier) {
                constexpr int n = 16 - barrier, at = m - barrier;
                StaticFor<at * 16 / n, (at + 1) * 16 / n>::run([&](auto d) { request(Int<slot>(), d); });
            }
        });
        if constexpr (G == 4) request_scales(Int<1 - P>());
        if constexpr (barrier >= 0) next_line();
    };
    auto superblock = [&](auto pp) { StaticFor<0, 8>::run([&](auto g) { group(g, pp); }); };
    for (;;) {
        superblock(Int<0>());
        if (--supers == 0) break;
        superblock(Int<1>());
        if (--supers == 0) break;
    }
    // The last superblock has read fragments of one that does not exist: nothing may be scheduled above the wait (main_loop of
    // gemm_i8.hip).  The last results need 18 wait states before a vector instruction reads them; the requests past the end have landed.
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    hold_accumulators<64>();
    __syncthreads();

    // ---- epilogue: 32 rows at a time through a private LDS region, then eight (bf16) or four consecutive columns per lane: whole
    // lines per request.  A lane beyond the matrix skips its store: through the stores of single columns, masked one by one, 2048 x 2176 x
    // 1024 took 18.7 us instead of 15.4.
    float* region = reinterpret_cast<float*>(smem_big) + wave * 32 * kLineEpiPitch;
    const int64_t row0 = m0 + wave_m * 128, col0 = n0 + wave_n * 128;
    StaticFor<0, 4>::run([&](auto ii) {
        constexpr int i = decltype(ii)::value;
        __builtin_amdgcn_sched_barrier(0);
        hold_accumulators<64>();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        StaticFor<0, 16>::run([&](auto qq) {                     // tile 4 i + q / 4, columns 8 (q % 4) + 4 half
            constexpr int q = decltype(qq)::value;
            *reinterpret_cast<v4i*>(region + lrow * kLineEpiPitch + 32 * (q >> 2) + 8 * (q & 3) + 4 * half) = read_acc<16 * i + q>();
        });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (a.c_is_f32) {
            const int cc = 4 * lrow;
            const int64_t left = a.N - (col0 + cc);
#pragma unroll
            for (int p = 0; p < 16; ++p) {
                const int rr = 2 * p + half;
                const v4f v = *reinterpret_cast<const v4f*>(region + rr * kLineEpiPitch + cc);
                float* dst = reinterpret_cast<float*>(a.C) + (row0 + 32 * i + rr) * a.ldc + col0 + cc;
                if (row0 + 32 * i + rr >= a.M || left <= 0) continue;
                if (left >= 4) {
                    __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(dst));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e < left) dst[e] = v[e];
                }
            }
        } else {
            const int cc = 8 * (lane & 15);
            const int64_t left = a.N - (col0 + cc);
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int rr = 4 * p + (lane >> 4);
                const v4f x = *reinterpret_cast<const v4f*>(region + rr * kLineEpiPitch + cc);
                const v4f y = *reinterpret_cast<const v4f*>(region + rr * kLineEpiPitch + cc + 4);
                const v4u w = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
                uint16_t* dst = reinterpret_cast<uint16_t*>(a.C) + (row0 + 32 * i + rr) * a.ldc + col0 + cc;
                if (row0 + 32 * i + rr >= a.M || left <= 0) continue;
                if (left >= 8) {
                    __builtin_nontemporal_store(w, reinterpret_cast<v4u*>(dst));
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (e < left) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
    });
}

}  // namespace

hipError_t launch_gemm_mx6(const Mx6GemmArgs& a, hipStream_t s) {
    if (a.M == 0 || a.N == 0) return hipSuccess;
    if (a.K % 128 != 0) return hipErrorInvalidValue;
    const int64_t big_m = (a.M + 255) / 256, big_n = (a.N + 255) / 256;
    const int64_t tiles_m = (a.M + 127) / 128, tiles_n = (a.N + 127) / 128;
    if (tiles_m * tiles_n > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int64_t c_bytes = a.c_is_f32 ? 4 : 2;
    // What the DMA kernels take: 16-byte stores need aligned rows of C.  Whole lines: K in superblocks of 384 code bytes, scale rows in
    // 16-byte chunks, the rows of a tile inside one buffer.
    const bool big = (a.ldc * c_bytes) % 16 == 0 && (reinterpret_cast<uintptr_t>(a.C) & 15u) == 0;
    const int64_t most = ((int64_t(1) << 32) - 1024) / 256;
    const bool lines = a.K > 0 && a.K % 512 == 0 && a.lda <= most && a.ldb <= most && a.ldsa <= most && a.ldsb <= most &&
                       a.ldsa % 16 == 0 && a.ldsb % 16 == 0 && (reinterpret_cast<uintptr_t>(a.SA) & 15u) == 0 &&
                       (reinterpret_cast<uintptr_t>(a.SB) & 15u) == 0;
    // In whole lines as soon as a compute unit would get two of the small tiles, where the product is long enough: about 10 us + 0.006
    // for each element of K as long as the 256 x 256 tiles fit the chip once, against 7 + 0.01 for up to two small tiles a compute unit,
    // less for narrow ones.  Small tiles against whole lines, tokens x out-features x in-features: 1024 x 4096 x 4096 (256 small tiles)
    // 31.5 us / 36.4, 2048 x 3072 x 4096 50.3 / 36.3, 768 x 14336 x 4096 77.1 / 38.2, 640 x 14336 x 8192 137 / 65; K = 2048: 33024 x 16
    // 23.9 / 24.2, 2048 x 2176 29.1 / 21.6; K = 1536: 33024 x 16 19.1 / 20.6, x 64 21.6 / 19.8; K = 1024: 2048 x 2176 17.9 / 15.4, 1040 x
    // 3712 15.2 / 15.2, 129 x 16640 14.5 / 15.2, 33024 x 16 13.7 / 16.7; K = 512: 2304 x 4096 (576 small tiles) 20.8 / 13.0, 384 x 14336
    // (336) 13.7 / 13.0, 1040 x 3712 (261) 11.1 / 13.6, 129 x 16640 10.5 / 13.3, 33024 x 16 8.6 / 13.1.
    // Other K: the eight-wavefront kernel where its tiles fill most of the chip; whole lines are as fast or faster than that at any K.
    const int64_t small_tiles = tiles_m * tiles_n;
    const bool long_enough = a.K >= 2048 || (a.N > 64 && (a.K >= 1536 || (a.M > 256 && (a.K >= 1024 || small_tiles > 320))));
    if (big && (big_m * big_n >= 192 || (lines && small_tiles > kComputeUnits && long_enough))) {
        static std::once_flag once;
        static hipError_t attr_result = hipSuccess;
        std::call_once(once, [&] {
            attr_result = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_mx6_big_kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, kBigLds);
            if (attr_result == hipSuccess)
                attr_result = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_mx6_lines_kernel),
                                                  hipFuncAttributeMaxDynamicSharedMemorySize, kLinesLds);
        });
        if (attr_result != hipSuccess) return attr_result;
        const dim3 grid((unsigned)(big_m * big_n));
        if (lines) hipLaunchKernelGGL(gemm_mx6_lines_kernel, grid, dim3(256), kLinesLds, s, a, (int)big_m, (int)big_n);
        else hipLaunchKernelGGL(gemm_mx6_big_kernel, grid, dim3(512), kBigLds, s, a, (int)big_m, (int)big_n);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(gemm_mx6_kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0, s, a, (int)tiles_n);
    return hipGetLastError();
}

}  // namespace halo
