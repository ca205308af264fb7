// Row transform kernels: right-hand Walsh-Hadamard rotation along the contiguous axis fused with the
// symmetric absmax INT8 quantiser (or with a plain bf16/fp32 store for the un-rotation of GEMM outputs).
//
// One wavefront owns one SEGMENT of 2^LOGSEG consecutive elements of a row and keeps it in registers:
// element index inside the segment = [chunk | lane (6 bits) | e], with the low LOGE bits (e) in
// consecutive registers (one 16-byte load per chunk), the next six bits across the 64 lanes, and the
// remaining high bits across chunks.  The butterflies therefore run
//      strides 1 .. EPL/2      in registers,
//      the next six strides    across lanes (DPP / ds_swizzle / ds_bpermute),
//      the highest strides     in registers again,
// i.e. in ascending stride order, every add/sub a separately rounded fp32 operation.
//
// Cross-lane stages: wave_ops.h.  They leave a sign, parity of (position & mask of the cross-lane stages run), which is folded
// into the 1/sqrt(d) factor at the end and costs nothing.
#pragma clang fp contract(off)

#include <algorithm>
#include <mutex>

#include "halo_internal.h"
#include "wave_ops.h"

namespace halo {
namespace {

constexpr float kRoundMagic = 12582912.0f;  // 1.5 * 2^23: adding it rounds |x| < 2^22 to an integer, ties to even

template <int VPL, int RB>
__device__ __forceinline__ void stage_in_regs(float (&v)[VPL]) {
    constexpr int H = 1 << RB;
#pragma unroll
    for (int r = 0; r < VPL; ++r) {
        if ((r & H) == 0) {
            const float a = v[r], b = v[r | H];
            v[r] = a + b;
            v[r | H] = a - b;
        }
    }
}

// Run stage number BIT (stride 2^BIT) of the segment-local FWHT if it is below log_block.
template <int VPL, int LOGE, int BIT>
__device__ __forceinline__ void fwht_stage(float (&v)[VPL], int log_block, int lane, int bperm_addr) {
    if (BIT < log_block) {
        if constexpr (BIT < LOGE) {
            stage_in_regs<VPL, BIT>(v);
        } else if constexpr (BIT < LOGE + 6) {
            stage_across_lanes<VPL, BIT - LOGE>(v, lane, bperm_addr);
        } else {
            stage_in_regs<VPL, BIT - 6>(v);
        }
    }
}

template <int VPL, int LOGE, int BIT, int LOGSEG>
struct FwhtStages {
    static __device__ __forceinline__ void run(float (&v)[VPL], int log_block, int lane, int bperm_addr) {
        fwht_stage<VPL, LOGE, BIT>(v, log_block, lane, bperm_addr);
        FwhtStages<VPL, LOGE, BIT + 1, LOGSEG>::run(v, log_block, lane, bperm_addr);
    }
};
template <int VPL, int LOGE, int LOGSEG>
struct FwhtStages<VPL, LOGE, LOGSEG, LOGSEG> {
    static __device__ __forceinline__ void run(float (&)[VPL], int, int, int) {}
};

// Per-wave geometry shared by the phases of the kernel.
struct RowCtx {
    int lane, bperm_addr;   // lane: the lane's position in the element order (wave_ops.h)
    int wave, seg;          // wavefront in the workgroup; segment of the row it owns
    float* xbuf;            // LDS exchange buffer [waves][values per lane / 4][64][4] (only with cross-wave stages)
    int64_t row, kbase;     // kbase: first element of this lane's chunk 0
    bool row_ok;
    bool f32;               // IN_F32_I32: this matrix holds fp32 (uniform over the workgroup)
};

// Quantising blocks of 4096: 1/sqrt(block) is a power of two, and the multiply by it (and the lanes' signs) is not made on every
// value but once, on the factor that quantises them, 127 / absmax or a power of two.  Scaling by a power of two is exact, so the
// codes are the same ones as long as nothing on the way leaves the normal range: kTiny < absmax < kHuge; otherwise every value
// is multiplied after all.  One vector instruction of some 22 (INT8) or 26 (MXFP6) per element in kernels that are bound by
// them: 4096 x 4096 to INT8 14.0 -> 13.5 us, 8192 x 4096 to MXFP6 32.4 -> 30.9.  (Blocks of 1024 and 256 are bound by their loads, and
// 3 % slower that way.)
template <int OUT, int LB>
constexpr bool kDeferNorm = (OUT == OUT_Q8 || OUT == OUT_MX6) && LB == 12;
constexpr float kTiny = 0x1p-100f, kHuge = 0x1p100f;
__device__ __forceinline__ bool may_defer(float amax) { return amax > kTiny && amax < kHuge; }

// Load one segment into registers, rotate it, apply the fold vector; returns the local absmax (quantising kernels but GIVEN_MAX).
// FAST: the row exists and the whole segment lies inside it, so nothing is bounds-checked.
// deferred: what the values are still to be multiplied by (kDeferNorm; the absmax is not), otherwise 1.
template <int LOGSEG, int IN, int OUT, bool FAST, int LB, int XS, int MAX>
__device__ __forceinline__ float row_phase1(const RowArgs& a, const RowCtx& x, float c_norm,
                                            float (&v)[1 << (LOGSEG - 6)], float& deferred) {
    constexpr int LOGE = (IN == IN_BF16) ? 3 : 2;
    constexpr int EPL = 1 << LOGE;
    constexpr int VPL = 1 << (LOGSEG - 6);
    constexpr int NCH = VPL / EPL;

    float pre = 1.0f;
    if constexpr (IN == IN_I32 || IN == IN_F32_I32) {
        if (IN == IN_F32_I32 && x.f32) pre = a.in_mul != 0.0f ? a.in_mul : 1.0f;      // x * 1.0f is x
        else if (x.row_ok && a.pre_scale) pre = a.pre_scale[x.row];
    }
    auto widen = [&](int32_t q) { return (IN == IN_F32_I32 && x.f32 ? __int_as_float(q) : (float)q) * pre; };
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int64_t k0 = x.kbase + (int64_t)c * 64 * EPL;
        if (FAST || (x.row_ok && k0 + EPL <= a.cols)) {
            if constexpr (IN == IN_BF16) {
                const uint4 q = *reinterpret_cast<const uint4*>(
                    reinterpret_cast<const uint16_t*>(a.in) + x.row * a.ld_in + k0);
                const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[c * EPL + 2 * i] = __uint_as_float(w[i] << 16);
                    v[c * EPL + 2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
                }
            } else if constexpr (IN == IN_F32) {
                const float4 q = *reinterpret_cast<const float4*>(
                    reinterpret_cast<const float*>(a.in) + x.row * a.ld_in + k0);
                v[c * EPL + 0] = q.x; v[c * EPL + 1] = q.y; v[c * EPL + 2] = q.z; v[c * EPL + 3] = q.w;
            } else {
                const int4 q = *reinterpret_cast<const int4*>(
                    reinterpret_cast<const int32_t*>(a.in) + x.row * a.ld_in + k0);
                v[c * EPL + 0] = widen(q.x); v[c * EPL + 1] = widen(q.y);
                v[c * EPL + 2] = widen(q.z); v[c * EPL + 3] = widen(q.w);
            }
        } else {
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                float t = 0.0f;
                if (x.row_ok && k0 + e < a.cols) {
                    if constexpr (IN == IN_BF16) {
                        t = __uint_as_float((uint32_t)(reinterpret_cast<const uint16_t*>(a.in)[x.row * a.ld_in + k0 + e]) << 16);
                    } else if constexpr (IN == IN_F32) {
                        t = reinterpret_cast<const float*>(a.in)[x.row * a.ld_in + k0 + e];
                    } else {
                        t = widen(reinterpret_cast<const int32_t*>(a.in)[x.row * a.ld_in + k0 + e]);
                    }
                }
                v[c * EPL + e] = t;
            }
        }
    }

    if constexpr (IN == IN_F32) {
        if (a.in_mul != 0.0f) {      // e.g. the 1/sqrt(block) of a left-hand rotation whose butterflies ran before
#pragma unroll
            for (int r = 0; r < VPL; ++r) v[r] *= a.in_mul;
        }
    }
    if constexpr (IN == IN_I32 || IN == IN_F32_I32) {
        if (a.post_scale && !(IN == IN_F32_I32 && x.f32)) {          // one more (tensor-wide) scale, applied after the per-row one
            const float post = *a.post_scale;
#pragma unroll
            for (int r = 0; r < VPL; ++r) v[r] *= post;
        }
    }

    // ---- rotate (LB >= 0: block size known at compile time, so the stage sequence is straight-line code)
    const int log_block = LB >= 0 ? LB : a.log_block;
    if (log_block > 0) {
        FwhtStages<VPL, LOGE, 0, LOGSEG>::run(v, log_block, x.lane, x.bperm_addr);
        if constexpr (XS > 0) {
            // Strides 2^LOGSEG .. 2^(LOGSEG+XS-1) pair up whole segments, i.e. wavefronts of this workgroup: each wavefront publishes its
            // registers in LDS and combines them with its partner's, the lower segment taking a+b and the upper one a-b (the lane
            // signs carried so far are the same in both), 16 bytes a lane at a time.  bf16 inputs, two strides: it publishes once
            // and also works out what its partner of the second one has after the first, one more add per value for one barrier
            // instead of three; blocks of 4096, quantising 2048 x 4096 9.5 -> 8.7 us, 1024 x 8192 9.7 -> 9.1.  32-bit inputs go a
            // round per stride: the un-rotations of 2048 x 4096 and 4096 x 4096 take 28.9 us in one launch so, and 28.9 with the
            // 4-byte accesses of before.
            static_assert(XS <= 2 && VPL % 4 == 0, "wavefronts of a block");
            float4* xb = reinterpret_cast<float4*>(x.xbuf) + x.lane;
            const float sg0 = x.seg & 1 ? -1.0f : 1.0f, sg1 = x.seg & 2 ? -1.0f : 1.0f;
            constexpr bool AT_ONCE = XS == 2 && IN == IN_BF16;
#pragma unroll
            for (int xs = 0; xs < (AT_ONCE ? 1 : XS); ++xs) {
                if (xs > 0) __syncthreads();        // everyone has read the previous round
#pragma unroll
                for (int r = 0; r < VPL; r += 4)
                    xb[(x.wave * VPL + r) * 16] = make_float4(v[r], v[r + 1], v[r + 2], v[r + 3]);
                __syncthreads();
                const float sg = xs == 0 ? sg0 : sg1;
#pragma unroll
                for (int r = 0; r < VPL; r += 4) {
                    const float4 p = xb[((x.wave ^ (1 << xs)) * VPL + r) * 16];
                    v[r] = __builtin_fmaf(v[r], sg, p.x);
                    v[r + 1] = __builtin_fmaf(v[r + 1], sg, p.y);
                    v[r + 2] = __builtin_fmaf(v[r + 2], sg, p.z);
                    v[r + 3] = __builtin_fmaf(v[r + 3], sg, p.w);
                    if constexpr (AT_ONCE) {
                        const float4 q = xb[((x.wave ^ 2) * VPL + r) * 16], o = xb[((x.wave ^ 3) * VPL + r) * 16];
                        v[r] = __builtin_fmaf(v[r], sg1, __builtin_fmaf(q.x, sg0, o.x));
                        v[r + 1] = __builtin_fmaf(v[r + 1], sg1, __builtin_fmaf(q.y, sg0, o.y));
                        v[r + 2] = __builtin_fmaf(v[r + 2], sg1, __builtin_fmaf(q.z, sg0, o.z));
                        v[r + 3] = __builtin_fmaf(v[r + 3], sg1, __builtin_fmaf(q.w, sg0, o.w));
                    }
                }
            }
        }
        // lanes whose (lane & mask) has odd parity hold negated values: the sign rides on the 1/sqrt(d) multiply
        int nlane_stages = log_block - LOGE;
        nlane_stages = nlane_stages < 0 ? 0 : (nlane_stages > 6 ? 6 : nlane_stages);
        const int mask = (1 << nlane_stages) - 1;
        const float sign_l = (__builtin_popcount(x.lane & mask) & 1) ? -1.0f : 1.0f;
        const float c_l = sign_l * c_norm;
        if (kDeferNorm<OUT, LB> && !a.fold) {                     // uniform
            deferred = c_l;
        } else {
#pragma unroll
            for (int r = 0; r < VPL; ++r) v[r] *= c_l;
        }
    }

    // ---- fold
    if (a.fold) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = x.kbase + (int64_t)c * 64 * EPL;
            if (FAST || k0 + EPL <= a.cols) {
#pragma unroll
                for (int i = 0; i < EPL / 4; ++i) {
                    const float4 f = *reinterpret_cast<const float4*>(a.fold + k0 + 4 * i);
                    v[c * EPL + 4 * i + 0] *= f.x; v[c * EPL + 4 * i + 1] *= f.y;
                    v[c * EPL + 4 * i + 2] *= f.z; v[c * EPL + 4 * i + 3] *= f.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (k0 + e < a.cols) v[c * EPL + e] *= a.fold[k0 + e];
            }
        }
    }

    float amax = 0.0f;
    if constexpr (OUT == OUT_Q8 && MAX != GIVEN_MAX) {
        // one v_max3_f32 with |.| source modifiers per pair of values (written out: the compiler's fmaxf chain takes
        // four instructions per pair), in two chains
        float amax2 = 0.0f;
#pragma unroll
        for (int r = 0; r < VPL; r += 4) {
            asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(amax) : "v"(v[r]), "v"(v[r + 1]));
            asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(amax2) : "v"(v[r + 2]), "v"(v[r + 3]));
        }
        amax = __builtin_fmaxf(amax, amax2);
        if (kDeferNorm<OUT, LB> && !a.fold) amax *= c_norm;
        amax = wave_max(amax, x.bperm_addr);
    }
    return amax;
}

// Quantise (inv_l = per-lane signed 127/absmax) or convert, and store the segment.
// MXFP6: inv_l is what the values are still to be multiplied by (kDeferNorm), or 1.
template <int LOGSEG, int IN, int OUT, bool FAST>
__device__ __forceinline__ void row_phase2(const RowArgs& a, const RowCtx& x, const float (&v)[1 << (LOGSEG - 6)],
                                           float inv_l) {
    constexpr int LOGE = (IN == IN_BF16) ? 3 : 2;
    constexpr int EPL = 1 << LOGE;
    constexpr int VPL = 1 << (LOGSEG - 6);
    constexpr int NCH = VPL / EPL;
    if constexpr (OUT == OUT_Q8) {
        int8_t* orow = reinterpret_cast<int8_t*>(a.out) + x.row * a.ld_out;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = x.kbase + (int64_t)c * 64 * EPL;
            uint32_t packed[EPL / 4];
#pragma unroll
            for (int i = 0; i < EPL / 4; ++i) {
                uint32_t b[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float t = v[c * EPL + 4 * i + e] * inv_l;
                    b[e] = __float_as_uint(t + kRoundMagic);
                }
                const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u);
                const uint32_t hi = __builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u);
                packed[i] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
            }
            if (FAST || (x.row_ok && k0 + EPL <= a.cols)) {
                if constexpr (EPL == 8) {
                    *reinterpret_cast<uint2*>(orow + k0) = make_uint2(packed[0], packed[1]);
                } else {
                    *reinterpret_cast<uint32_t*>(orow + k0) = packed[0];
                }
            } else if (x.row_ok) {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (k0 + e < a.cols) orow[k0 + e] = (int8_t)((packed[e / 4] >> (8 * (e & 3))) & 0xFF);
            }
        }
    } else if constexpr (OUT == OUT_MX6) {
        // Microscaling FP6: the four lanes of a quad hold one block of 32 consecutive elements.  Shared scale
        // 2^(floor(log2(block absmax)) - 4) (E8M0), elements rounded to E3M2 (ties to even mantissa, saturating at 28),
        // eight 6-bit codes per lane packed least-significant first; the quad's 24 bytes leave as 8 + 4 + 8 + 4.
        static_assert(EPL == 8, "MXFP6 output takes bf16 input");
        unsigned char* orow = reinterpret_cast<unsigned char*>(a.out) + x.row * a.ld_out;
        const int j = x.lane & 3;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = x.kbase + (int64_t)c * 64 * EPL;
            float bm = 0.0f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) bm = __builtin_fmaxf(bm, fabsf(v[c * EPL + e]));
            bm = __builtin_fmaxf(bm, lane_xor<0>(bm, x.bperm_addr));
            bm = __builtin_fmaxf(bm, lane_xor<1>(bm, x.bperm_addr)) * fabsf(inv_l);
            int shared = (int)(__float_as_uint(bm) >> 23) - 127 - 4;
            shared = shared < -127 ? -127 : shared;               // the upper clamp cannot bind: exponent <= 127 - 4
            if (!(bm > 0.0f)) shared = 0;
            // Round |x| 2^-shared to E3M2 with one addition: 2^(e + 21), e >= -2 the element's exponent, has units of 2^(e - 2) in
            // its last place, so that the sum's low bits are the element in those units (four of them to a binade, ties to even)
            // and its exponent field gives the rest of the code; below 2^-2 the units stay 2^-4.  No code has a negative zero:
            // up to 2^-5 the element rounds to 0.  Ten VALU instructions an element, which bound this kernel; sixteen, with integer
            // rounding and a path for subnormals, took 38.5 us at 8192 x 4096 instead of 36.4, 22.8 instead of 20.6 at 4096 x 4096.
            float scale = __uint_as_float((uint32_t)(127 - shared) << 23);               // 2^-shared, 3 <= exponent field <= 254
            float w[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) w[e] = v[c * EPL + e];
            if (__all(bm == 0.0f || may_defer(bm))) {
                scale *= inv_l;
            } else {
#pragma unroll
                for (int e = 0; e < EPL; ++e) w[e] *= inv_l;
            }
            uint32_t code[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                const float xs = w[e] * scale;
                const float ax = __builtin_fminf(fabsf(xs), 28.0f);
                const float pow2 = __uint_as_float(__float_as_uint(__builtin_fmaxf(ax, 0.25f)) & 0x7F800000u);
                const uint32_t u = __float_as_uint(__builtin_fmaf(pow2, 2097152.0f, ax));
                code[e] = (u & 15u) + (u >> 21) + (xs < -0.03125f ? 32u - 584u : 0u - 584u);     // 584 = 4 (125 + 21)
            }
            const uint32_t w0 = code[0] | (code[1] << 6) | (code[2] << 12) | (code[3] << 18) | (code[4] << 24) | (code[5] << 30);
            const uint32_t w1 = (code[5] >> 2) | (code[6] << 4) | (code[7] << 10);
            const uint32_t nb_w0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)w0, 0xB1, 0xF, 0xF, true);   // of position ^ 1 (j even: j + 1)
            if (FAST || (x.row_ok && k0 + EPL <= a.cols)) {
                unsigned char* blk = orow + (k0 >> 5) * 24;          // k0 >> 5 is the same for the four lanes of the quad
                if ((j & 1) == 0) {
                    uint32_t* dst = reinterpret_cast<uint32_t*>(blk + 12 * (j >> 1));
                    dst[0] = w0;
                    dst[1] = w1 | (nb_w0 << 16);
                } else {
                    *reinterpret_cast<uint32_t*>(blk + 8 + 12 * (j >> 1)) = (w0 >> 16) | (w1 << 16);
                }
                if (j == 0) a.mx_scales[x.row * a.ld_mx_scales + (k0 >> 5)] = (uint8_t)(shared + 127);
            }
        }
    } else if constexpr (OUT == OUT_BF16) {
        uint16_t* orow = reinterpret_cast<uint16_t*>(a.out) + x.row * a.ld_out;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = x.kbase + (int64_t)c * 64 * EPL;
            uint32_t packed[EPL / 2];
#pragma unroll
            for (int i = 0; i < EPL / 2; ++i)
                packed[i] = pack_bf16x2(v[c * EPL + 2 * i], v[c * EPL + 2 * i + 1]);
            if (FAST || (x.row_ok && k0 + EPL <= a.cols)) {
                if constexpr (EPL == 8) {
                    *reinterpret_cast<uint4*>(orow + k0) = make_uint4(packed[0], packed[1], packed[2], packed[3]);
                } else {
                    *reinterpret_cast<uint2*>(orow + k0) = make_uint2(packed[0], packed[1]);
                }
            } else if (x.row_ok) {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (k0 + e < a.cols) orow[k0 + e] = (uint16_t)(packed[e / 2] >> (16 * (e & 1)));
            }
        }
    } else {
        float* orow = reinterpret_cast<float*>(a.out) + x.row * a.ld_out;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = x.kbase + (int64_t)c * 64 * EPL;
            if (FAST || (x.row_ok && k0 + EPL <= a.cols)) {
#pragma unroll
                for (int i = 0; i < EPL / 4; ++i)
                    *reinterpret_cast<float4*>(orow + k0 + 4 * i) =
                        make_float4(v[c * EPL + 4 * i], v[c * EPL + 4 * i + 1], v[c * EPL + 4 * i + 2], v[c * EPL + 4 * i + 3]);
            } else if (x.row_ok) {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (k0 + e < a.cols) orow[k0 + e] = v[c * EPL + e];
            }
        }
    }
}

// LB: log2 of the Hadamard block when it is 0 (no rotation), LOGSEG (block = segment) or 9; -1 = read it at run time.
// XS: number of butterfly stages that span wavefronts (Hadamard block = 2^(LOGSEG+XS) elements = 2^XS segments).
template <int LOGSEG, int IN, int OUT, int LB, int XS, int MAX>
__device__ __forceinline__ void row_transform(RowArgs& a, int segs, int rows_per_wg, float c_norm, unsigned blocks1) {
    constexpr int LOGE = (IN == IN_BF16) ? 3 : 2;
    constexpr int EPL = 1 << LOGE;            // consecutive elements per lane per chunk
    constexpr int VPL = 1 << (LOGSEG - 6);    // values per lane
    constexpr int SEG = 1 << LOGSEG;

    __shared__ float s_amax[16];
    extern __shared__ __align__(16) float s_xbuf[];

    const int wave = threadIdx.x >> 6;
    const int seg = wave % segs;
    const int row_local = wave / segs;
    RowCtx x;
    x.wave = wave;
    x.seg = seg;
    x.xbuf = s_xbuf;
    x.lane = position_of_lane(threadIdx.x & 63);
    x.bperm_addr = ((threadIdx.x & 63) ^ 32) << 2;
    unsigned block = blockIdx.x;
    x.f32 = block < blocks1;
    if (block >= blocks1) {          // the second matrix of a batched launch
        block -= blocks1;
        a.in = a.in2; a.pre_scale = a.pre_scale2; a.out = a.out2; a.out_scale = a.out_scale2; a.rows = a.rows2;
        if constexpr (MAX == GIVEN_MAX) {
            if (a.given_amax2) { a.given_amax = a.given_amax2; a.given_parts = a.given_parts2; }
        }
        if (a.post_scale2) a.post_scale = a.post_scale2;
    }
    x.row = (int64_t)block * rows_per_wg + row_local;
    x.row_ok = x.row < a.rows;
    x.kbase = (int64_t)seg * SEG + (int64_t)x.lane * EPL;
    const bool fast = x.row_ok && ((int64_t)(seg + 1) * SEG <= a.cols);   // uniform over the wavefront

    // A block that is the segment divides the row: a wavefront has a whole segment or, past the last row, nothing.  Without a
    // guarded path the bf16 kernels fit the registers that four (4096) and eight or seven wavefronts (2048) of a SIMD leave, with none
    // in scratch memory; a bound on the registers alone left 3 to 8 of them there.  8192 x 14336 in blocks of 2048, quantised to
    // INT8: 82 us with neither, 69 with the bound, 67 so; 4096 x 8192 in blocks of 4096 23.8, 23.0, 21.2.  Shorter segments need no more
    // registers than they have; their guarded path stays (with 1024 it is 1 % faster).
    constexpr bool WHOLE = LB >= 11 && LB == LOGSEG;
    float given = 0.0f;
    if constexpr (MAX == GIVEN_MAX) given = part_of_given<kRowGivenLoads>(a.given_amax, a.given_parts);      // on their way with the row
    float v[VPL];
    float amax = 0.0f, deferred = 1.0f;
    if constexpr (WHOLE) {
        if (fast) amax = row_phase1<LOGSEG, IN, OUT, true, LB, XS, MAX>(a, x, c_norm, v, deferred);
    } else {
        amax = fast ? row_phase1<LOGSEG, IN, OUT, true, LB, XS, MAX>(a, x, c_norm, v, deferred)
                    : row_phase1<LOGSEG, IN, OUT, false, LB, XS, MAX>(a, x, c_norm, v, deferred);
    }

    float inv_l = 0.0f;
    if constexpr (OUT == OUT_Q8) {
        if constexpr (MAX == GIVEN_MAX) {
            amax = given_max(given, s_amax);
        } else if constexpr (MAX == MAX_ONLY) {
            amax = workgroup_max(amax, s_amax);
            if (threadIdx.x == 0) a.out_scale[block] = amax;
            return;
        } else if (segs > 1) {
            if (x.lane == 0) s_amax[wave] = amax;
            __syncthreads();
            const int w0 = row_local * segs;
            float t = s_amax[w0];
            for (int i = 1; i < segs; ++i) t = fmaxf(t, s_amax[w0 + i]);
            amax = t;
        }
        const bool nz = amax > 0.0f;
        inv_l = nz ? 127.0f / amax : 0.0f;
        if (x.row_ok && seg == 0 && x.lane == 0) a.out_scale[x.row] = nz ? amax / 127.0f : 1.0f;
        if constexpr (kDeferNorm<OUT, LB>) {
            if (may_defer(amax)) {                        // uniform over the wavefront
                inv_l *= deferred;
            } else {
#pragma unroll
                for (int r = 0; r < VPL; ++r) v[r] *= deferred;
            }
        }
    }
    if constexpr (OUT == OUT_MX6) inv_l = deferred;
    if (fast) row_phase2<LOGSEG, IN, OUT, true>(a, x, v, inv_l);
    else if constexpr (!WHOLE) row_phase2<LOGSEG, IN, OUT, false>(a, x, v, inv_l);
}

template <int LOGSEG, int IN, int OUT, int LB, int XS = 0>
__global__ void __launch_bounds__(LOGSEG >= 11 ? 512 : 1024)
row_transform_kernel(RowArgs a, int segs, int rows_per_wg, float c_norm, unsigned blocks1) {
    row_transform<LOGSEG, IN, OUT, LB, XS, OWN_MAX>(a, segs, rows_per_wg, c_norm, blocks1);
}

// One scale per tensor, in kernels of its own: as branches of the kernel above it lengthened every INT8 quantiser, by 0.1 us for the 512
// x 1024 W and 256 x 1024 X of a small level-2 step (level 2, 256 x 640 x 720, fp32 out: 33.2 us with the branches, 32.9 without).
template <int LOGSEG, int IN, int MAX, int LB, int XS = 0>
__global__ void __launch_bounds__(LOGSEG >= 11 ? 512 : 1024)
row_tensor_kernel(RowArgs a, int segs, int rows_per_wg, float c_norm, unsigned blocks1) {
    row_transform<LOGSEG, IN, OUT_Q8, LB, XS, MAX>(a, segs, rows_per_wg, c_norm, blocks1);
}

template <int LOGSEG, int IN, int OUT, int MAX, int LB, int XS = 0>
constexpr auto row_kernel() {
    if constexpr (MAX == OWN_MAX) return row_transform_kernel<LOGSEG, IN, OUT, LB, XS>;
    else return row_tensor_kernel<LOGSEG, IN, MAX, LB, XS>;
}

// How a launch cuts its rows: segments of 2^logseg elements, `stages` butterfly stages across wavefronts.
struct RowShape {
    int logseg, segs, stages;
    int rows_per_wg() const { return segs >= 4 || segs == 0 ? 1 : 4 / segs; }
    int threads() const { return 64 * segs * rows_per_wg(); }
};

// Workgroups of a launch, of the first matrix and of both.
struct RowGrid {
    int64_t blocks1, blocks;
    RowGrid(const RowArgs& a, int rows_per_wg)
        : blocks1((a.rows + rows_per_wg - 1) / rows_per_wg), blocks(blocks1 + (a.rows2 + rows_per_wg - 1) / rows_per_wg) {}
    // MAX_ONLY writes one value per workgroup
    void parts(int64_t* out) const {
        if (out) { out[0] = blocks1; out[1] = blocks - blocks1; }
    }
};

// Hadamard block of 2^(10+XS) elements handled by 2^XS wavefronts of 1024 elements each: four times the
// wavefronts of the one-wavefront-per-block layout and a quarter of the registers, at the price of XS round trips
// through LDS.  It pays when there are too few rows to fill the machine otherwise.
template <int IN, int OUT, int MAX, int XS>
hipError_t launch_split(const RowArgs& a, const RowShape& shape, hipStream_t s, int64_t* parts) {
    constexpr int LOGSEG = 10;
    const int threads = shape.threads(), rows_per_wg = shape.rows_per_wg();
    const RowGrid g(a, rows_per_wg);
    g.parts(parts);
    const float c_norm = (float)(1.0 / sqrt((double)(int64_t(1) << a.log_block)));
    const size_t lds = (size_t)(threads / 64) * (1 << (LOGSEG - 6)) * 64 * sizeof(float);
    constexpr auto kern = row_kernel<LOGSEG, IN, OUT, MAX, LOGSEG + XS, XS>();
    hipLaunchKernelGGL(kern, dim3((unsigned)g.blocks), dim3(threads), lds, s, a, shape.segs, rows_per_wg, c_norm, (unsigned)g.blocks1);
    return hipGetLastError();
}

template <int LOGSEG, int IN, int OUT, int MAX>
hipError_t launch_one(const RowArgs& a, const RowShape& shape, hipStream_t s, int64_t* parts) {
    const int threads = shape.threads(), rows_per_wg = shape.rows_per_wg();
    const RowGrid g(a, rows_per_wg);
    g.parts(parts);
    const float c_norm = a.log_block > 0 ? (float)(1.0 / sqrt((double)(int64_t(1) << a.log_block))) : 1.0f;
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)g.blocks), dim3(threads), 0, s, a, shape.segs, rows_per_wg, c_norm, (unsigned)g.blocks1);
        return hipGetLastError();
    };
    if (a.log_block == 0) {
        if constexpr (IN == IN_F32_I32) return hipErrorInvalidValue;      // only the paired un-rotation, which has a block
        else return launch(row_kernel<LOGSEG, IN, OUT, MAX, 0>());
    }
    if constexpr (IN == IN_BF16 && OUT == OUT_Q8 && LOGSEG == 10) {
        if (a.log_block == 9) return launch(row_kernel<LOGSEG, IN, OUT, MAX, 9>());
    }
    if (a.log_block == LOGSEG) return launch(row_kernel<LOGSEG, IN, OUT, MAX, LOGSEG>());
    return launch(row_kernel<LOGSEG, IN, OUT, MAX, -1>());
}

// logseg == 0: no shape fits.
template <int IN, int OUT>
RowShape row_shape(const RowArgs& a) {
    // Split blocks of 2048 / 4096 over 2 / 4 wavefronts (measured): the 32-bit-input un-rotation gains at every size
    // for 4096-blocks (5.7 vs 5.2 TB/s at 32768 rows, 12.7 vs 16.0 us at 2048 rows); the others, and 2048-blocks of the paired
    // un-rotation, when whole rows would leave the 1024 SIMDs with fewer than four wavefronts each (level-2 backward, 2048
    // in-features, 256 tokens by 256 22.6 -> 21.9 us, 1024 by 2048 51.6 -> 51.0, 4096 by 512 90.1 either way).
    if ((a.log_block == 11 || a.log_block == 12) && a.cols % 1024 == 0 && a.cols <= 16384) {
        const int64_t wavefronts_unsplit = (a.rows + a.rows2) * (a.cols >> a.log_block);
        const bool few = wavefronts_unsplit < 4096;
        const bool want = IN == IN_I32 ? a.log_block == 12 : IN == IN_F32_I32 ? a.log_block == 12 || few : few;
        if (want) return {10, (int)(a.cols >> 10), a.log_block - 10};
    }
    // Segment = max(Hadamard block, 512), grown until the row fits the workgroup (16 waves, 8 from 2048 up).  The INT8 quantiser of bf16
    // rows is bound by how much a compute unit has on its way: with blocks up to 512, segments of 1024, two loads per lane, are the
    // faster ones where a row has more than three of them and there are rows for all compute units (512 against 1024: 4096 x 2304 in
    // blocks of 256 11.35 us / 11.31, x 1280 7.2 / 8.0; 4096 x 3584 in blocks of 512 13.3 / 12.0, 8192 x 5632 40.5 / 32.1; 4096 x 5696 in
    // blocks of 64 20.7 / 17.6).  With few rows a wavefront's time counts, and that is longer: 16 x 5632 3.4 / 4.2, 256 x 5632 3.6 / 4.4,
    // 1024 x 3136 5.4 / 5.6, 768 x 4608 5.3 / 5.6, 512 x 5632 4.9 / 5.2, 256 x 7168 4.0 / 4.2; beyond the line 2048 x 3136 8.2 / 8.2, 1536 x
    // 3584 7.1 / 6.6, 1024 x 4608 6.2 / 6.0 (1536 x 4608 is an exception, 7.4 / 8.1), 768 x 5120 6.4 / 5.7, 640 x 5632 6.0 / 5.8, 512 x 7168
    // 5.7 / 5.2.  The un-rotations have 4-byte inputs, the MXFP6 quantiser more to do with a value, and 512 is the faster one for both
    // throughout.
    int logseg = a.log_block < 9 ? 9 : a.log_block;
    if (IN == IN_BF16 && OUT == OUT_Q8 && logseg == 9 && a.cols > 3072 && (a.rows + a.rows2) * (a.cols - 2048) >= 1 << 21) logseg = 10;
    if (a.log_block == 0) {
        // no rotation: any segmentation is valid; 1024-element segments keep register use low
        logseg = a.cols <= 512 ? 9 : 10;
    }
    for (;; ++logseg) {
        if (logseg > 12) return {0, 0, 0};
        const int64_t segs = (a.cols + (int64_t(1) << logseg) - 1) >> logseg;
        if (segs <= (logseg >= 11 ? 8 : 16)) return {logseg, (int)segs, 0};
    }
}

template <int IN, int OUT, int MAX = OWN_MAX>
hipError_t launch_by_seg(const RowArgs& a, hipStream_t s, int64_t* parts = nullptr) {
    const RowShape shape = row_shape<IN, OUT>(a);
    if (shape.stages == 1) return launch_split<IN, OUT, MAX, 1>(a, shape, s, parts);
    if (shape.stages == 2) return launch_split<IN, OUT, MAX, 2>(a, shape, s, parts);
    switch (shape.logseg) {
        case 9: return launch_one<9, IN, OUT, MAX>(a, shape, s, parts);
        case 10: return launch_one<10, IN, OUT, MAX>(a, shape, s, parts);
        case 11: return launch_one<11, IN, OUT, MAX>(a, shape, s, parts);
        case 12: return launch_one<12, IN, OUT, MAX>(a, shape, s, parts);
        default: return hipErrorInvalidValue;
    }
}

// The end of a left+right un-rotation (see halo_internal.h).  Workgroup = 2^TOP wavefronts; wavefront t owns row
// blk * hb + t * 256 + q of one right-hand block of 2^LOGSEG columns, hb = 256 << TOP: exactly the rows that the top TOP
// strides of the left-hand rotation (256, 512, ...) combine.  Stage st pairs wavefront t with t ^ 2^st through LDS (the
// lower row takes a + b, the upper one a - b), ascending; then the wavefront has its row of the left-rotated matrix in
// registers, in the layout of the row kernel, and goes on as that kernel does.
// TOP == 5 (segments up to 2048 columns): the 32 rows sit two to a wavefront, rows t * 256 + q and (t + 16) * 256 + q of the
// block of 8192; the first four of the five strides go through LDS as before, for both rows, and the last one (4096 rows)
// pairs the wavefront's own two rows in registers.
template <int LOGSEG, int OUT, int TOP>
__global__ void __launch_bounds__(TOP >= 5 ? 1024 : (64 << TOP), (LOGSEG >= 12 || TOP >= 5) ? 4 : 8)
row_left_top_kernel(RowArgs a, int segs, float c_norm) {
    constexpr int LOGE = 2, EPL = 4;
    constexpr int VPL = 1 << (LOGSEG - 6);
    constexpr int NCH = VPL / EPL;
    constexpr int SEG = 1 << LOGSEG;
    constexpr int NR = TOP >= 5 ? 2 : 1;                    // rows per wavefront
    constexpr int XT = TOP >= 5 ? 4 : TOP;                  // strides that go through LDS
    static_assert(TOP <= 5 && (TOP < 5 || LOGSEG <= 11), "32 rows of 4096 columns do not fit a compute unit");
    extern __shared__ __align__(16) float s_exch[];        // exchange buffer of the stages across wavefronts

    const int lane = position_of_lane(threadIdx.x & 63), wave = threadIdx.x >> 6;
    const int64_t g = (int64_t)blockIdx.x / segs;                 // group of 2^TOP rows: g = blk * 256 + q
    const int seg = (int)((int64_t)blockIdx.x % segs);
    const int64_t row0 = ((g >> 8) << (8 + TOP)) + ((int64_t)wave << 8) + (g & 255);
    const int64_t kbase = (int64_t)seg * SEG + (int64_t)lane * EPL;

    float v[NR][VPL];
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        const float* src = reinterpret_cast<const float*>(a.in) + (row0 + (int64_t)n * 4096) * a.ld_in + kbase;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const float4 q = *reinterpret_cast<const float4*>(src + c * 64 * EPL);
            v[n][c * EPL + 0] = q.x; v[n][c * EPL + 1] = q.y; v[n][c * EPL + 2] = q.z; v[n][c * EPL + 3] = q.w;
        }
    }
    // Exchange buffer: [wavefront][value / 4][lane][4] (16-byte LDS accesses), HALF values per wavefront at a time so that
    // two workgroups fit one compute unit's LDS and one of them can load while the other exchanges.
    constexpr int HALF = VPL > 16 ? VPL / 2 : VPL;
    float4* xb = reinterpret_cast<float4*>(s_exch);
    bool first_round = true;
#pragma unroll
    for (int st = 0; st < XT; ++st) {
        const float sg = (wave >> st) & 1 ? -1.0f : 1.0f;      // lower row a + b, upper row a - b, one exact product each
        const int pw = wave ^ (1 << st);
#pragma unroll
        for (int n = 0; n < NR; ++n) {
#pragma unroll
            for (int h0 = 0; h0 < VPL; h0 += HALF) {
                if (!first_round) __syncthreads();   // everyone has read the previous round
                first_round = false;
#pragma unroll
                for (int r = 0; r < HALF; r += 4)
                    xb[(wave * (HALF / 4) + r / 4) * 64 + lane] =
                        make_float4(v[n][h0 + r], v[n][h0 + r + 1], v[n][h0 + r + 2], v[n][h0 + r + 3]);
                __syncthreads();
#pragma unroll
                for (int r = 0; r < HALF; r += 4) {
                    const float4 p = xb[(pw * (HALF / 4) + r / 4) * 64 + lane];
                    v[n][h0 + r + 0] = __builtin_fmaf(v[n][h0 + r + 0], sg, p.x);
                    v[n][h0 + r + 1] = __builtin_fmaf(v[n][h0 + r + 1], sg, p.y);
                    v[n][h0 + r + 2] = __builtin_fmaf(v[n][h0 + r + 2], sg, p.z);
                    v[n][h0 + r + 3] = __builtin_fmaf(v[n][h0 + r + 3], sg, p.w);
                }
            }
        }
    }
    if constexpr (NR == 2) {               // the last stride: the wavefront's own two rows
#pragma unroll
        for (int r = 0; r < VPL; ++r) {
            const float x = v[0][r], y = v[NR - 1][r];
            v[0][r] = x + y;
            v[NR - 1][r] = x - y;
        }
    }
    const int bperm_addr = ((threadIdx.x & 63) ^ 32) << 2;
    const float c_l = (__builtin_popcount(lane) & 1) ? -c_norm : c_norm;     // the sign the lane stages leave behind
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        if (a.in_mul != 0.0f) {
#pragma unroll
            for (int r = 0; r < VPL; ++r) v[n][r] *= a.in_mul;
        }
        // right-hand un-rotation of the row (block = segment), as in row_phase1
        FwhtStages<VPL, LOGE, 0, LOGSEG>::run(v[n], LOGSEG, lane, bperm_addr);
#pragma unroll
        for (int r = 0; r < VPL; ++r) v[n][r] *= c_l;

        RowCtx x;
        x.lane = lane; x.bperm_addr = bperm_addr; x.wave = wave; x.seg = seg; x.xbuf = s_exch;
        x.row = row0 + (int64_t)n * 4096; x.kbase = kbase; x.row_ok = true;
        row_phase2<LOGSEG, IN_F32, OUT, true>(a, x, v[n], 0.0f);
    }
}

template <int LOGSEG, int OUT, int TOP>
hipError_t launch_left_top(const RowArgs& a, hipStream_t s) {
    constexpr int VPL = 1 << (LOGSEG - 6);
    constexpr int kWaves = TOP >= 5 ? 16 : (1 << TOP);
    constexpr int kLds = kWaves * (VPL > 16 ? VPL / 2 : VPL) * 64 * (int)sizeof(float);
    static std::once_flag once;
    static hipError_t attr_result = hipSuccess;
    auto kern = row_left_top_kernel<LOGSEG, OUT, TOP>;
    std::call_once(once, [&] {
        if (kLds > 64 * 1024)
            attr_result = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    });
    if (attr_result != hipSuccess) return attr_result;
    const int segs = (int)(a.cols >> LOGSEG);
    const int64_t blocks = (a.rows >> TOP) * segs;
    if (blocks <= 0 || blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const float c_norm = (float)(1.0 / sqrt((double)(int64_t(1) << LOGSEG)));
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * kWaves), kLds, s, a, segs, c_norm);
    return hipGetLastError();
}

template <int LOGSEG, int OUT>
hipError_t launch_left_top_by_top(const RowArgs& a, hipStream_t s) {
    switch (a.left_top) {
        case 1: return launch_left_top<LOGSEG, OUT, 1>(a, s);
        case 2: return launch_left_top<LOGSEG, OUT, 2>(a, s);
        case 3: return launch_left_top<LOGSEG, OUT, 3>(a, s);
        case 4: return launch_left_top<LOGSEG, OUT, 4>(a, s);
        case 5:
            if constexpr (LOGSEG <= 11) return launch_left_top<LOGSEG, OUT, 5>(a, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

template <int OUT>
hipError_t launch_left_top_by_seg(const RowArgs& a, hipStream_t s) {
    switch (a.log_block) {
        case 9: return launch_left_top_by_top<9, OUT>(a, s);
        case 10: return launch_left_top_by_top<10, OUT>(a, s);
        case 11: return launch_left_top_by_top<11, OUT>(a, s);
        case 12: return launch_left_top_by_top<12, OUT>(a, s);
        default: return hipErrorInvalidValue;
    }
}

// The row quantiser behind the top TOP strides of a left-hand rotation (halo_internal.h): a wavefront holds the same 1024
// columns of the 2^TOP rows that those strides combine, so the strides are adds in registers, and the fp32 intermediate is
// not written and read once more for them.  Bound by memory, 4 + 1 bytes an element, as the plain row quantiser is;
// every load, the fold vector's too, is requested under one branch (4096 x 4096: with a branch per row and fold element by element
// 20.5 us, so 16).
template <int TOP>
__global__ void __launch_bounds__(1024)
row_top_quant_kernel(RowArgs a, int segs, int groups_per_wg, int low) {
    constexpr int NR = 1 << TOP, VPL = 16;
    __shared__ float s_amax[16][NR];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int seg = wave % segs, local = wave / segs;
    const int64_t g = (int64_t)blockIdx.x * groups_per_wg + local;
    const bool ok = g < (a.rows >> TOP);
    const int64_t row0 = ((g >> low) << (low + TOP)) + (g & ((int64_t(1) << low) - 1));
    const int64_t kbase = (int64_t)seg * 1024 + lane * 4;
    const bool fast = ok && (int64_t)(seg + 1) * 1024 <= a.cols;
    float v[NR][VPL], f[VPL];
    const float* const src = reinterpret_cast<const float*>(a.in) + row0 * a.ld_in + kbase;
    const int64_t next = a.ld_in << low;
    if (fast) {                            // one branch around all loads
#pragma unroll
        for (int n = 0; n < NR; ++n)
#pragma unroll
            for (int c = 0; c < VPL; c += 4) {
                const float4 q = *reinterpret_cast<const float4*>(src + n * next + c * 64);
                v[n][c] = q.x; v[n][c + 1] = q.y; v[n][c + 2] = q.z; v[n][c + 3] = q.w;
            }
        if (a.fold) {
#pragma unroll
            for (int c = 0; c < VPL; c += 4) {
                const float4 q = *reinterpret_cast<const float4*>(a.fold + kbase + c * 64);
                f[c] = q.x; f[c + 1] = q.y; f[c + 2] = q.z; f[c + 3] = q.w;
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < VPL; ++c) {
            const int k = (c >> 2) * 256 + (c & 3);
            const bool in = ok && kbase + k < a.cols;
#pragma unroll
            for (int n = 0; n < NR; ++n) v[n][c] = in ? src[n * next + k] : 0.0f;
            f[c] = in && a.fold ? a.fold[kbase + k] : 1.0f;
        }
    }
#pragma unroll
    for (int h = 1; h < NR; h <<= 1)
#pragma unroll
        for (int n = 0; n < NR; ++n)
            if ((n & h) == 0) {
#pragma unroll
                for (int c = 0; c < VPL; ++c) {
                    const float x = v[n][c], y = v[n | h][c];
                    v[n][c] = x + y;
                    v[n | h][c] = x - y;
                }
            }
#pragma unroll
    for (int n = 0; n < NR; ++n)
#pragma unroll
        for (int c = 0; c < VPL; ++c) v[n][c] *= a.in_mul;
    if (a.fold) {
#pragma unroll
        for (int n = 0; n < NR; ++n)
#pragma unroll
            for (int c = 0; c < VPL; ++c) v[n][c] *= f[c];
    }
    const int bperm_addr = (lane ^ 32) << 2;
    float amax[NR];
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        float m0 = 0.0f, m1 = 0.0f;
#pragma unroll
        for (int c = 0; c < VPL; c += 4) {
            asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m0) : "v"(v[n][c]), "v"(v[n][c + 1]));
            asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m1) : "v"(v[n][c + 2]), "v"(v[n][c + 3]));
        }
        amax[n] = wave_max(__builtin_fmaxf(m0, m1), bperm_addr);
    }
    if (segs > 1) {
        if (lane == 0) {
#pragma unroll
            for (int n = 0; n < NR; ++n) s_amax[wave][n] = amax[n];
        }
        __syncthreads();
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            amax[n] = s_amax[local * segs][n];
            for (int i = 1; i < segs; ++i) amax[n] = fmaxf(amax[n], s_amax[local * segs + i][n]);
        }
    }
    RowCtx x;
    x.lane = lane; x.bperm_addr = bperm_addr; x.wave = wave; x.seg = seg; x.xbuf = nullptr;
    x.kbase = kbase; x.row_ok = ok;
#pragma unroll
    for (int n = 0; n < NR; ++n) {
        const bool nz = amax[n] > 0.0f;
        const float inv = nz ? 127.0f / amax[n] : 0.0f;
        x.row = row0 + ((int64_t)n << low);
        if (ok && seg == 0 && lane == 0) a.out_scale[x.row] = nz ? amax[n] / 127.0f : 1.0f;
        if (fast) row_phase2<10, IN_F32, OUT_Q8, true>(a, x, v[n], inv);
        else row_phase2<10, IN_F32, OUT_Q8, false>(a, x, v[n], inv);
    }
}

}  // namespace

hipError_t launch_row_top_quant(const RowArgs& a, int low, hipStream_t s) {
    if (a.rows == 0 || a.cols == 0) return hipSuccess;
    if (!row_top_quant_ok(a.cols, a.left_top) || a.log_block != 0 || a.kron_m != 0 || a.rows2 != 0 || low < 0 ||
        a.rows % (int64_t(1) << (low + a.left_top)) != 0)
        return hipErrorInvalidValue;
    const int segs = (int)((a.cols + 1023) >> 10), groups_per_wg = segs >= 4 ? 1 : 4 / segs;
    const int64_t groups = a.rows >> a.left_top, blocks = (groups + groups_per_wg - 1) / groups_per_wg;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    auto* kern = a.left_top == 1 ? row_top_quant_kernel<1> : row_top_quant_kernel<2>;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * segs * groups_per_wg), 0, s, a, segs, groups_per_wg, low);
    return hipGetLastError();
}

hipError_t launch_row_left_top(const RowArgs& a, OutKind out, hipStream_t s) {
    if (a.kron_m != 0 || a.fold || a.rows2 != 0 || !row_left_top_ok(a.rows, a.cols, a.log_block, a.left_top))
        return hipErrorInvalidValue;
    if (out == OUT_BF16) return launch_left_top_by_seg<OUT_BF16>(a, s);
    if (out == OUT_F32) return launch_left_top_by_seg<OUT_F32>(a, s);
    return hipErrorInvalidValue;
}

int64_t max_given_parts(const RowArgs& a, InKind in) {
    int threads = 0;
    if (a.kron_m != 0) threads = (int)(a.cols / 28);
    else if (in == IN_BF16) threads = row_shape<IN_BF16, OUT_Q8>(a).threads();
    else if (in == IN_F32) threads = row_shape<IN_F32, OUT_Q8>(a).threads();
    return (int64_t)kRowGivenLoads * std::min(threads, 256);
}

// Its kernels, and launch_row_max's, are made last: which kernels come first in the object decides where they lie, and these kernels, which
// run straight through some 10 KB of instructions, depend on that by a few per cent (X and W of 2048 x 4096 x 4096, the same
// instructions: 21.0 us at one address, 20.1 at one 4 KB further on; 20.3 in this order, 20.5 before there were any of those).
static hipError_t launch_row_given(const RowArgs& a, InKind in, hipStream_t s);

hipError_t launch_row_transform(const RowArgs& a, InKind in, OutKind out, hipStream_t s) {
    if ((a.rows == 0 && a.rows2 == 0) || a.cols == 0) return hipSuccess;
    if (a.kron_m != 0) return out == OUT_MX6 || in == IN_F32_I32 ? hipErrorInvalidValue : launch_row_kron(a, in, out, s);
    if (a.cols > kMaxRowCols || a.log_block > 12) return hipErrorInvalidValue;
    if (a.given_amax) return out == OUT_Q8 ? launch_row_given(a, in, s) : hipErrorInvalidValue;
    if (in == IN_BF16 && out == OUT_Q8) return launch_by_seg<IN_BF16, OUT_Q8>(a, s);
    if (in == IN_F32 && out == OUT_Q8) return launch_by_seg<IN_F32, OUT_Q8>(a, s);
    if (in == IN_I32 && out == OUT_BF16) return launch_by_seg<IN_I32, OUT_BF16>(a, s);
    if (in == IN_I32 && out == OUT_F32) return launch_by_seg<IN_I32, OUT_F32>(a, s);
    if (in == IN_F32_I32 && a.rows2 > 0 && out == OUT_BF16) return launch_by_seg<IN_F32_I32, OUT_BF16>(a, s);
    if (in == IN_F32_I32 && a.rows2 > 0 && out == OUT_F32) return launch_by_seg<IN_F32_I32, OUT_F32>(a, s);
    if (in == IN_F32 && out == OUT_BF16) return launch_by_seg<IN_F32, OUT_BF16>(a, s);
    if (in == IN_F32 && out == OUT_F32) return launch_by_seg<IN_F32, OUT_F32>(a, s);
    if (in == IN_BF16 && out == OUT_MX6) return a.cols % 32 == 0 ? launch_by_seg<IN_BF16, OUT_MX6>(a, s) : hipErrorInvalidValue;
    return hipErrorInvalidValue;
}

hipError_t launch_row_max(const RowArgs& a, InKind in, int64_t* parts, hipStream_t s) {
    if (a.rows == 0 || a.cols == 0 || a.given_amax) return hipErrorInvalidValue;
    if (a.kron_m != 0) return launch_row_kron_max(a, in, parts, s);
    if (a.cols > kMaxRowCols || a.log_block > 12) return hipErrorInvalidValue;
    if (in == IN_BF16) return launch_by_seg<IN_BF16, OUT_Q8, MAX_ONLY>(a, s, parts);
    if (in == IN_F32) return launch_by_seg<IN_F32, OUT_Q8, MAX_ONLY>(a, s, parts);
    return hipErrorInvalidValue;
}

static hipError_t launch_row_given(const RowArgs& a, InKind in, hipStream_t s) {
    if (bad_given_parts(a, in)) return hipErrorInvalidValue;
    if (in == IN_BF16) return launch_by_seg<IN_BF16, OUT_Q8, GIVEN_MAX>(a, s);
    if (in == IN_F32) return launch_by_seg<IN_F32, OUT_Q8, GIVEN_MAX>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace halo
