// What the matrix kernels share: the workgroup -> tile map, global -> LDS transfers, and accumulators that are named in the text of
// inline assembly.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gemm_offsets.h"

namespace halo {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

#define HALO_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

template <int V>
using Int = std::integral_constant<int, V>;

// f(Int<0>), f(Int<1>), ... f(Int<N-1>): loops whose index has to be a constant expression (immediate offsets).
template <int I, int N>
struct StaticFor {
    template <class F>
    static __device__ __forceinline__ void run(const F& f) {
        if constexpr (I < N) {
            f(Int<I>());
            StaticFor<I + 1, N>::run(f);
        }
    }
};

// Consecutive workgroup ids go to different XCDs (8 per chip): give every XCD a contiguous range of tile
// numbers, and walk tiles in groups of GROUP tile-rows so that one XCD's resident tiles share A and B panels in
// its L2 (measured on an 8192^3 product: 22 % L2 misses with this map, 51 % without the XCD step).  `bid` counts
// from the first workgroup of the product: for the second product of a paired launch that rotates the XCD numbers by
// (first product's workgroups) % 8, which still hands every hardware XCD one contiguous range of tile numbers.
template <int GROUP>
__device__ __forceinline__ void tile_of_block(int bid, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    const int ntiles = tiles_m * tiles_n;
    const int xcd = bid & 7, q = bid >> 3;
    const int base = ntiles >> 3, rem = ntiles & 7;
    const int pid = xcd * base + (xcd < rem ? xcd : rem) + q;
    const int per_group = GROUP * tiles_n;
    const int group = pid / per_group;
    const int first_m = group * GROUP;
    const int gsize = (tiles_m - first_m) < GROUP ? (tiles_m - first_m) : GROUP;
    const int in_group = pid % per_group;
    tile_m = first_m + in_group % gsize;
    tile_n = in_group / gsize;
}

// 16 bytes per lane, buffer offset voff -> LDS (lds + 16 * lane).  Offsets past the buffer's end deliver zeros.
// m0 is a reserved register and cannot be declared as overwritten; the build fails if the compiler uses it in these kernels.
constexpr uint32_t kBufferBytes = 0xFFFFFF00u;
static_assert(kOutside >= kBufferBytes, "kOutside is past the end");
__device__ __forceinline__ void dma16(uint32_t voff, const v4u& buffer, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voff), "s"(buffer), "s"(lds)
                 : "memory");
}
__device__ __forceinline__ v4u make_buffer(const void* base) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    return (v4u){(uint32_t)p, (uint32_t)(p >> 32) & 0xFFFFu, kBufferBytes, 0x00020000u};
}
__device__ __forceinline__ void advance(v4u& buffer, int64_t bytes) {
    const uint64_t p = (((uint64_t)buffer[1] << 32) | buffer[0]) + (uint64_t)bytes;
    buffer[0] = (uint32_t)p;
    buffer[1] = (uint32_t)(p >> 32);
}

// The accumulators are NOT variables: register tile t of a wavefront is the accumulation registers a[4 t .. 4 t + 3], named
// in the text of the assembly below.  (As variables they fill the whole accumulation half of the register file, and every
// branch or epilogue made the compiler copy or spill them.)  hold_accumulators() tells the compiler that they are taken:
// nothing that the compiler keeps can live in them across one, and one stands at every wait and before every row or column
// of tiles of the epilogues.  Between two holds the compiler could still put a short-lived value there: the build reads the
// generated code and fails if these kernels touch an accumulation register outside this assembly, or use scratch memory.
#define HALO_A8(n) "a" #n "0", "a" #n "1", "a" #n "2", "a" #n "3", "a" #n "4", "a" #n "5", "a" #n "6", "a" #n "7", "a" #n "8", "a" #n "9"
#define HALO_ACCUMULATORS                                                                                               \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", HALO_A8(1), HALO_A8(2), HALO_A8(3), HALO_A8(4), HALO_A8(5), \
        HALO_A8(6), HALO_A8(7), HALO_A8(8), HALO_A8(9), HALO_A8(10), HALO_A8(11), HALO_A8(12), HALO_A8(13), HALO_A8(14),    \
        HALO_A8(15), HALO_A8(16), HALO_A8(17), HALO_A8(18), HALO_A8(19), HALO_A8(20), HALO_A8(21), HALO_A8(22),             \
        HALO_A8(23), HALO_A8(24), "a250", "a251", "a252", "a253", "a254", "a255"
#define HALO_ACCUMULATORS_128                                                                                           \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", HALO_A8(1), HALO_A8(2), HALO_A8(3), HALO_A8(4), HALO_A8(5), \
        HALO_A8(6), HALO_A8(7), HALO_A8(8), HALO_A8(9), HALO_A8(10), HALO_A8(11), "a120", "a121", "a122", "a123", "a124",   \
        "a125", "a126", "a127"
#define HALO_ACCUMULATORS_64                                                                                            \
    "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", HALO_A8(1), HALO_A8(2), HALO_A8(3), HALO_A8(4), HALO_A8(5), \
        "a60", "a61", "a62", "a63"
template <int TILES>
__device__ __forceinline__ void hold_accumulators() {
    if constexpr (TILES > 32) asm volatile("" ::: HALO_ACCUMULATORS);
    else if constexpr (TILES > 16) asm volatile("" ::: HALO_ACCUMULATORS_128);
    else asm volatile("" ::: HALO_ACCUMULATORS_64);
}
template <int T>
__device__ __forceinline__ void clear_acc() {
    asm volatile("v_accvgpr_write_b32 a[%0], 0\n\tv_accvgpr_write_b32 a[%1], 0\n\tv_accvgpr_write_b32 a[%2], 0\n\t"
                 "v_accvgpr_write_b32 a[%3], 0" ::"n"(4 * T), "n"(4 * T + 1), "n"(4 * T + 2), "n"(4 * T + 3));
}
template <int T>
__device__ __forceinline__ v4i read_acc() {
    v4i v;
    int x, y, z, w;
    asm volatile("v_accvgpr_read_b32 %0, a[%4]\n\tv_accvgpr_read_b32 %1, a[%5]\n\tv_accvgpr_read_b32 %2, a[%6]\n\t"
                 "v_accvgpr_read_b32 %3, a[%7]"
                 : "=v"(x), "=v"(y), "=v"(z), "=v"(w)
                 : "n"(4 * T), "n"(4 * T + 1), "n"(4 * T + 2), "n"(4 * T + 3));
    v = (v4i){x, y, z, w};
    return v;
}
template <int T>
__device__ __forceinline__ void write_acc(const v4i& v) {
    asm volatile("v_accvgpr_write_b32 a[%4], %0\n\tv_accvgpr_write_b32 a[%5], %1\n\tv_accvgpr_write_b32 a[%6], %2\n\t"
                 "v_accvgpr_write_b32 a[%7], %3" ::"v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "n"(4 * T), "n"(4 * T + 1),
                 "n"(4 * T + 2), "n"(4 * T + 3));
}

}  // namespace halo
