// Internal declarations shared by the HIP translation units of libhalo (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_plan.h"
#include "halo.h"

namespace halo {

// IN_F32_I32: the first matrix of a batched launch (rows2 > 0) holds fp32 and the second int32.
enum InKind { IN_BF16 = 0, IN_F32 = 1, IN_I32 = 2, IN_F32_I32 = 3 };
enum OutKind { OUT_Q8 = 0, OUT_BF16 = 1, OUT_F32 = 2, OUT_MX6 = 3 };
// Where the row quantisers' absmax comes from.  OWN_MAX: the row's own.  One scale per tensor takes two launches: MAX_ONLY writes the
// largest |value| of each workgroup's rows and no codes, GIVEN_MAX quantises with the largest of those.
enum RowMax { OWN_MAX, MAX_ONLY, GIVEN_MAX };

// ---- row transform: [pre-scale] -> right-hand FWHT -> [fold] -> {absmax+INT8 | bf16 | fp32} ----
struct RowArgs {
    const void* in;
    int64_t ld_in;
    int64_t rows, cols;
    const float* pre_scale;  // int32 only: per-row multiplier, may be null
    const float* fold;       // per-column multiplier, may be null
    void* out;
    int64_t ld_out;
    float* out_scale;        // OUT_Q8 only
    int log_block;           // log2 of the Hadamard block, 0 = no rotation
    int kron_m;              // 0, or 28: the block is 28 * 2^log_block elements, rotated by H_{2^log_block} (x) H_28
    float in_mul;            // fp32 only: every element is multiplied by this once when it is loaded; 0 = no multiply
    int left_top;            // launch_row_left_top only: number of top strides of the left-hand rotation still to run (1..5)
    // One scale per tensor (OUT_Q8 only): the largest of the given_parts values at given_amax (device memory; launch_row_max,
    // tensor_max_parts) replaces the row's own absmax.  post_scale (IN_I32 only, device scalar) is multiplied in after pre_scale.
    // Both apply to both matrices of a batched launch.
    int given_parts;
    const float* given_amax;
    const float* post_scale;
    // OUT_MX6 only (bf16 input, cols a multiple of 32): `out` receives the packed FP6 E3M2 codes (24 bytes per block of
    // 32 elements, ld_out in BYTES per row), mx_scales the E8M0 scale bytes [rows x cols/32] with ld_mx_scales bytes per row.
    uint8_t* mx_scales;
    int64_t ld_mx_scales;
    // Optional second matrix handled by the same launch (same cols, leading dimensions, fold and block; its own
    // row count and buffers): rows2 == 0 means none.  Saves one launch ramp/tail when two independent tensors get
    // the same treatment (X and W in the forward pass, the two accumulators of the backward pass).
    int64_t rows2;
    const void* in2;
    const float* pre_scale2;
    void* out2;
    float* out_scale2;
    const float* given_amax2;    // the second matrix's own given_amax / post_scale; null: those of the first
    const float* post_scale2;
    int given_parts2;
};
// Largest row length the row kernels accept.
constexpr int64_t kMaxRowCols = 32768;
hipError_t launch_row_transform(const RowArgs& a, InKind in, OutKind out, hipStream_t s);
// The first of the two launches of a quantiser with one scale per tensor (bf16 or fp32 in): no codes, but the largest |rotated value| of
// the rows of each workgroup, written to out_scale (and out_scale2).  parts[0] (parts[1]) are set to how many those are, at most one
// per row.
hipError_t launch_row_max(const RowArgs& a, InKind in, int64_t* parts, hipStream_t s);
// Kronecker blocks (kron_m == 28): true if a row of `cols` elements can be rotated in blocks of `block` = 28 * 2^n
// elements (64 <= 2^n <= 512, block divides cols, cols <= 14336).  launch_row_transform forwards such launches.
// The end of a left+right un-rotation in one kernel.  `in` is fp32 [rows x cols] on which all strides of a left-hand
// rotation of block 256 << left_top have run except the top left_top ones; the kernel runs those (the 2^left_top rows
// they mix sit in the wavefronts of one workgroup and meet in LDS), multiplies by in_mul, un-rotates each row in blocks
// of 2^log_block and stores bf16 / fp32.  row_left_top_ok: the shapes it takes.
hipError_t launch_row_left_top(const RowArgs& a, OutKind out, hipStream_t s);
// The row quantiser (fp32 in, no right-hand rotation) behind the top strides of a left-hand rotation: rows r, r + 2^low,
// ... r + (2^left_top - 1) 2^low of a block of 2^(low + left_top) rows are combined, multiplied by in_mul (and fold), and
// quantised.  row_top_quant_ok: the shapes it takes.
inline bool row_top_quant_ok(int64_t cols, int left_top) { return left_top >= 1 && left_top <= 2 && cols <= 16 * 1024; }
hipError_t launch_row_top_quant(const RowArgs& a, int low, hipStream_t s);
bool row_kron_shape_ok(int64_t cols, int64_t block);
hipError_t launch_row_kron(const RowArgs& a, InKind in, OutKind out, hipStream_t s);
hipError_t launch_row_kron_max(const RowArgs& a, InKind in, int64_t* parts, hipStream_t s);

// ---- column-wise absmax quantiser with transposed output (E^T)_Q ----
struct ColQuantArgs {
    const void* in;          // bf16 [rows x cols]
    int64_t ld_in;
    int64_t rows, cols;
    const float* fold;       // per-row multiplier, may be null
    int8_t* out_q;           // [cols x rows]
    int64_t ld_q;
    float* out_scale;        // [cols]
    float* amax_ws;          // scratch: column absmax accumulated as bit patterns [cols], or partial maxima (see ColFwhtArgs)
};

// ---- left-hand (strided axis) FWHT: all stages of block 2^log_block, ascending, possibly several passes ----
// The first pass works on blocks of consecutive rows where it can (left_first_pass), the others are strided.  out is fp32; in
// may be out when it is fp32 too.  tmp (fp32 [rows x ld_tmp], may be out) carries what is between two passes.
struct ColFwhtArgs {
    const void* in;
    InKind in_kind;          // IN_BF16, IN_F32 or IN_I32
    int64_t ld_in;
    void* out;               // fp32
    int64_t ld_out;
    float* tmp;
    int64_t ld_tmp;
    int64_t rows, cols;
    int log_block;
    // IN_I32 input (accumulators of a product): element (r, k) enters as (float(in[r,k]) * row_scale[r]) * post_scale[0]
    // (either pointer may be null).  first_stage: the strides below 2^first_stage have been applied already.  skip_norm:
    // leave the 1/sqrt(block) multiply to the caller.
    const float* row_scale;
    const float* post_scale;
    int first_stage;
    int skip_norm;
    // only_low > 0 (7 .. 11, with columns 6 .. 11; first_stage 0): the strides below 2^only_low, in one pass; the caller runs the others.
    int only_low;
    // columns != null (bf16 input, only_low > 0): the pass also works for that column quantiser of the same matrix.  A block that is
    // all of the rows: it writes its codes and scales.  Otherwise it writes the absolute maxima of each block of 2^only_low rows
    // to columns->amax_ws [rows >> only_low][cols], for launch_col_quant_t_ready.
    const ColQuantArgs* columns;
};
hipError_t launch_col_fwht(const ColFwhtArgs& a, hipStream_t s);

hipError_t launch_col_quant_t(const ColQuantArgs& a, hipStream_t s);
// The same with `parts` vectors of the columns' partial maxima already in a.amax_ws [parts x cols] (ColFwhtArgs::columns).
hipError_t launch_col_quant_t_ready(const ColQuantArgs& a, int parts, hipStream_t s);
// The same with one absmax for every column instead of the columns' own, the largest of `parts` values in device memory: the
// tensor-wide scale.
hipError_t launch_col_quant_t_given(const ColQuantArgs& a, const float* given_amax, int parts, hipStream_t s);
// What the kernels that take a tensor's absmax in parts are given: the parts as launch_row_max left them, or, where there are more
// than `most`, reduced to one value at `out` first by a launch of their own (in2, n2, out2: of a second tensor in the same launch, which
// is made for both if one of them has too many).  Returns the parts by changing in / n (in2 / n2).
hipError_t tensor_max_parts(const float*& in, int64_t& n, float* out, const float*& in2, int64_t& n2, float* out2, int64_t most,
                            hipStream_t s);
// `most`: what the threads of a workgroup read in so many loads each, all on their way with the first loads of what is quantised; 256
// threads for the kernels that quantise tiles.  Read in a loop at the end of the row quantiser, behind the rotation, 2048 and 4096 parts
// cost more than the launch that reduces them (X and W of 2048 x 4096 x 4096: 23.4 us, the reduction 4.7 + 18.9; so 19.2 without one).
// Calls, reduced / read at the end / so: forward 4096 x 512 x 512 17.4 us / 18.4 / 15.2, 2048 x 4096 x 4096 61.5 / 62.8 / 58.2;
// transposed codes of 4096 x 4096 18.1 / 21.1 / 16.0, of 4096 x 64 12.9 / 13.9 / 10.4.  Loads a thread: rows of 2048 x 4096 with 4 (so
// reduced) 16.7, with 8 14.8, with 16 15.4; tiles of 4096 x 4096 with 8 (reduced) 18.6, with 16 16.0.
constexpr int kRowGivenLoads = 8, kTileGivenLoads = 16;
constexpr int64_t kMaxTileGivenParts = kTileGivenLoads * 256;
int64_t max_given_parts(const RowArgs& a, InKind in);
inline bool bad_given_parts(const RowArgs& a, InKind in) {
    const int64_t most = max_given_parts(a, in);
    return a.given_parts <= 0 || a.given_parts > most || (a.given_amax2 && (a.given_parts2 <= 0 || a.given_parts2 > most));
}

// ---- both quantisations of E for the backward pass from one tiling (rows for E_X, transposed columns for G) ----
struct DualQuantArgs {
    const void* in;          // bf16 [rows x cols]
    int64_t ld_in;
    int64_t rows, cols;
    const float* fold_c;     // per-column multiplier of the row-wise quantisation (saved weight scales), may be null
    const float* fold_r;     // per-row multiplier of the column-wise quantisation (saved activation scales), may be null
    int8_t* out_q;           // [rows x cols]
    int64_t ld_q;
    float* row_scale;        // [rows]
    int8_t* out_qt;          // [cols x rows]
    int64_t ld_qt;
    float* col_scale;        // [cols]
    float* amax_ws;          // dual_quant_workspace_floats(rows, cols) floats of scratch
};
size_t dual_quant_workspace_floats(int64_t rows, int64_t cols);
hipError_t launch_dual_quant(const DualQuantArgs& a, hipStream_t s);
// The same with one absmax for all rows and columns, the largest of `parts` values in device memory, and no fold vectors: the codes of
// the two outputs are the same ones.  amax_ws is not used.
hipError_t launch_dual_quant_given(const DualQuantArgs& a, const float* given_amax, int parts, hipStream_t s);
// The same with the partial maxima in a file-scope device array instead of a.amax_ws (which is ignored): no allocation,
// no workspace argument.  Sizes whose partial maxima exceed kStaticScratchBytes are refused by the caller.
constexpr size_t kStaticScratchBytes = size_t(8) << 20;
hipError_t launch_dual_quant_static(DualQuantArgs a, hipStream_t s);

// ---- INT8 GEMM ----
constexpr int kMaxLowRank = 64;
hipError_t launch_gemm_i8(const GemmArgs& a, hipStream_t s);
hipError_t launch_gemm_i8_pair(const GemmArgs& a1, const GemmArgs& a2, hipStream_t s);
// True if `cfg` names a tile configuration that can run a product with reduction length K.
bool gemm_config_valid(int cfg, int64_t K);
// 256 workgroups x 8 wavefronts x iters x 32 MFMAs on the 4 KB of operand bytes at `operands`.
hipError_t launch_mfma_i8_probe(const int8_t* operands, int iters, int32_t* sink, hipStream_t s);

// ---- low-rank side branch (LoRA adapters next to the quantised products) ----
// out fp32 [rows x rank] = in bf16 [rows x K] times the thin bf16 operand: [rank x K] (its transpose is applied), or
// [K x rank] with k_major.  K a multiple of 64.
hipError_t launch_lr_down(const void* in, int64_t ld_in, const void* thin, int k_major, int64_t ld_b, float* out, int64_t rows,
                          int64_t K, int rank, hipStream_t s);
// out = big^T small: big bf16 [rows x wide], small fp32 [rows x rank] dense; out fp32 [wide x rank], or its transpose
// [rank x wide] with transpose_out.  part: lr_grad_workspace_floats(rows, wide, rank) floats of scratch.
struct LrGradArgs {
    const void* big;
    int64_t ld_big;
    const float* small;
    float* out;
    int transpose_out;
    float* part;
    int64_t wide;
};
size_t lr_grad_workspace_floats(int64_t rows, int64_t wide, int rank);
// The rotated forms of the thin operands of the E_X epilogue:  u_rot fp32 [m x rank] = the TRANSPOSE of u bf16
// [rank x m] with every row rotated in blocks of block_m (2^n, or 28 * 2^n; <= 1: only widened), and sm_rot fp32
// [b x rank] = sm fp32 [b x rank] with every column rotated in blocks of block_b (a power of two).  Either pair may be null.
struct LrRotArgs {
    const void* u;
    float* u_rot;
    int64_t m, block_m;
    const float* sm;
    float* sm_rot;
    int64_t b, block_b;
};
bool lr_row_fwht_shape_ok(int64_t cols, int64_t block);
bool lr_col_fwht_shape_ok(int64_t rows, int64_t block);
// Everything small of the backward pass of the low-rank branch in two launches: the gradient products a and b (either or
// both may be null), then the sums over their token ranges together with the rotations `rot` (may be null).
hipError_t launch_lr_backward_small(const LrGradArgs* a, const LrGradArgs* b, int64_t rows, int rank, const LrRotArgs* rot,
                                    hipStream_t s);

// ---- MXFP6 GEMM: C[M x N] = A[M x K] B[N x K]^T on packed E3M2 codes with one E8M0 scale per 32 elements along K ----
struct Mx6GemmArgs {
    const uint8_t* A; int64_t lda;          // packed codes, bytes per row
    const uint8_t* SA; int64_t ldsa;        // scale bytes, bytes per row
    const uint8_t* B; int64_t ldb;
    const uint8_t* SB; int64_t ldsb;
    int64_t M, N, K;                        // K a multiple of 128
    void* C; int c_is_f32; int64_t ldc;     // elements
};
hipError_t launch_gemm_mx6(const Mx6GemmArgs& a, hipStream_t s);

// fp32 -> bf16, round to nearest even, on the hardware conversion (v_cvt_pk_bf16_f32: two values per instruction).
typedef __bf16 halo_bf16x2 __attribute__((ext_vector_type(2)));
typedef float halo_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const halo_f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, halo_bf16x2));
}
__device__ __forceinline__ uint16_t bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

}  // namespace halo
