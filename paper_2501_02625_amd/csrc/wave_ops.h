// Butterflies and maxima across the lanes of a wavefront, for the row kernels.
//
// A lane's POSITION is its place in the order of the elements.  Positions are lanes, but inside every eight lanes the upper four
// are taken in reverse (position_of_lane, its own inverse): positions that differ in bit 2 then sit in lanes l and l ^ 7, so that
// each of the strides 1, 2, 4, 8 is one DPP operand of the add.  (Numbered straight, stride 4 went through ds_swizzle: an LDS
// instruction and a wait for every value.)  Addresses, signs and LDS slots all go by position.
//
// A stage runs x <- x + s * partner(x) with s = +1 in the lane holding the lower element and s = -1 in the other one: one
// rounded add or subtract (the product is exact).  The lower lane gets a + b; the upper one b - a, the exact negation of the
// wanted difference (fp32 add, subtract and fma with an exact product are sign-symmetric under round-to-nearest-even).  Two
// elements that meet in a later butterfly differ in one index bit only, so they carry the same accumulated sign and every later
// stage is again exact up to that common sign: parity of the position bits run so far, folded into the 1/sqrt(d) multiply.
#pragma once

#include <hip/hip_runtime.h>

namespace halo {

__device__ __forceinline__ int position_of_lane(int lane) { return (lane & 4) ? lane ^ 3 : lane; }

// The value of the lane whose position differs in bit J.  bperm_addr: (lane ^ 32) * 4 of the lane itself.
template <int J>
__device__ __forceinline__ float lane_xor(float x, int bperm_addr) {
    const int xi = __float_as_int(x);
    int r;
    if constexpr (J == 0) {
        r = __builtin_amdgcn_mov_dpp(xi, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    } else if constexpr (J == 1) {
        r = __builtin_amdgcn_mov_dpp(xi, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    } else if constexpr (J == 2) {
        r = __builtin_amdgcn_mov_dpp(xi, 0x141, 0xF, 0xF, true);  // row_half_mirror: lane ^ 7
    } else if constexpr (J == 3) {
        r = __builtin_amdgcn_mov_dpp(xi, 0x128, 0xF, 0xF, true);  // row_ror:8 == xor 8 inside a row of 16
    } else if constexpr (J == 4) {
        r = __builtin_amdgcn_ds_swizzle(xi, 0x401F);              // bit mode: xor 16
    } else {
        r = __builtin_amdgcn_ds_bpermute(bperm_addr, xi);         // lane ^ 32
    }
    return __int_as_float(r);
}

__device__ __forceinline__ float wave_max(float x, int bperm_addr) {
    x = __builtin_fmaxf(x, lane_xor<0>(x, bperm_addr));
    x = __builtin_fmaxf(x, lane_xor<1>(x, bperm_addr));
    x = __builtin_fmaxf(x, lane_xor<2>(x, bperm_addr));
    x = __builtin_fmaxf(x, lane_xor<3>(x, bperm_addr));
    x = __builtin_fmaxf(x, lane_xor<4>(x, bperm_addr));
    x = __builtin_fmaxf(x, lane_xor<5>(x, bperm_addr));
    return x;
}

// The largest of the workgroup's values, for every thread.  m: the largest of the thread's wavefront, non-negative; s_red: a float of
// LDS per wavefront, of which there are at most 16, that nothing else uses.
__device__ __forceinline__ float workgroup_max(float m, float* s_red) {
    const int waves = (int)(blockDim.x + 63) >> 6, i = (int)(threadIdx.x & 15);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = s_red[i < waves ? i : 0];
    m = __builtin_fmaxf(m, lane_xor<0>(m, 0));
    m = __builtin_fmaxf(m, lane_xor<1>(m, 0));
    m = __builtin_fmaxf(m, lane_xor<2>(m, 0));
    return __builtin_fmaxf(m, lane_xor<3>(m, 0));
}
// One scale per tensor: the largest of n non-negative values in memory, 1 <= n <= LOADS * threads.  Here a thread's part of them,
// without a loop or a branch, so that the loads are on their way together with whatever is loaded next; then the workgroup's.
template <int LOADS>
__device__ __forceinline__ float part_of_given(const float* p, int n) {
    float m = 0.0f;
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        const int i = (int)(threadIdx.x + u * blockDim.x);
        m = __builtin_fmaxf(m, p[i < n ? i : n - 1]);
    }
    return m;
}
__device__ __forceinline__ float given_max(float part, float* s_red) {
    return workgroup_max(wave_max(part, (int)((threadIdx.x & 63) ^ 32) << 2), s_red);
}

// Four  x <- x + s * partner(x)  in one asm block: v_fmac_f32 with the partner read through DPP.  The leading s_nop supplies
// the two wait states a DPP read needs after a vector write of the same register, whatever the compiler placed before the
// block; inside the block every register is read and written by one instruction.
#define HALO_FMAC_DPP4(X0, X1, X2, X3, S, CTRL)                                                                  \
    asm volatile("s_nop 1\n\t"                                                                                   \
                 "v_fmac_f32_dpp %0, %0, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %1, %1, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %2, %2, %4 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %3, %3, %4 " CTRL " row_mask:0xf bank_mask:0xf"                                   \
                 : "+v"(X0), "+v"(X1), "+v"(X2), "+v"(X3)                                                         \
                 : "v"(S))
#define HALO_FMAC_DPP8(X, R, S, CTRL)                                                                            \
    asm volatile("s_nop 1\n\t"                                                                                   \
                 "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                              \
                 "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf"                                   \
                 : "+v"(X[R]), "+v"(X[R + 1]), "+v"(X[R + 2]), "+v"(X[R + 3]), "+v"(X[R + 4]), "+v"(X[R + 5]),     \
                   "+v"(X[R + 6]), "+v"(X[R + 7])                                                                 \
                 : "v"(S))

// The stage that pairs positions differing in bit J, on N values per lane (a multiple of 4).
template <int N, int J>
__device__ __forceinline__ void stage_across_lanes(float (&v)[N], int position, int bperm_addr) {
    static_assert(N % 4 == 0, "values come in fours");
    const float s = ((position >> J) & 1) ? -1.0f : 1.0f;
    if constexpr (J < 4) {
#pragma unroll
        for (int r = 0; r + 8 <= N; r += 8) {
            if constexpr (J == 0) HALO_FMAC_DPP8(v, r, s, "quad_perm:[1,0,3,2]");
            else if constexpr (J == 1) HALO_FMAC_DPP8(v, r, s, "quad_perm:[2,3,0,1]");
            else if constexpr (J == 2) HALO_FMAC_DPP8(v, r, s, "row_half_mirror");
            else HALO_FMAC_DPP8(v, r, s, "row_ror:8");
        }
        if constexpr (N % 8 != 0) {
            constexpr int r = N - 4;
            if constexpr (J == 0) HALO_FMAC_DPP4(v[r], v[r + 1], v[r + 2], v[r + 3], s, "quad_perm:[1,0,3,2]");
            else if constexpr (J == 1) HALO_FMAC_DPP4(v[r], v[r + 1], v[r + 2], v[r + 3], s, "quad_perm:[2,3,0,1]");
            else if constexpr (J == 2) HALO_FMAC_DPP4(v[r], v[r + 1], v[r + 2], v[r + 3], s, "row_half_mirror");
            else HALO_FMAC_DPP4(v[r], v[r + 1], v[r + 2], v[r + 3], s, "row_ror:8");
        }
    } else {
#pragma unroll
        for (int r = 0; r < N; ++r) v[r] = __builtin_fmaf(lane_xor<J>(v[r], bperm_addr), s, v[r]);
    }
}

}  // namespace halo
