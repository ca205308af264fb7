// Where the INT8 GEMM kernels fetch a K-strided B from: plain integer functions, for the kernels and for a host program that
// walks every request against the size of the operand.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define HALO_HOST_DEVICE __attribute__((host, device, always_inline)) inline
#else
#define HALO_HOST_DEVICE inline
#endif

namespace halo {

// A buffer offset past the end of every buffer descriptor: the request delivers zeros and touches no memory.
constexpr uint32_t kOutside = 0xFFFFFFF0u;

// Chunk swizzle of a K-major row of BN bytes: distinct for the rows 0-7 and 16-23 (+ 8, + 32 ...) that one half-wavefront
// reads, where rows of 128 (64) bytes already alternate between the two halves (go round the four quarters) of the banks.
// Linear in the bits of the row.
template <int BN>
HALO_HOST_DEVICE constexpr int kmajor_swizzle(int row) {
    return BN == 256   ? (2 * (row & 7)) | ((row >> 4) & 1)
           : BN == 128 ? ((row >> 1) & 3) | (((row >> 4) & 1) << 2)
                       : ((row >> 2) & 1) | (((row >> 4) & 1) << 1);
}

// One request of a wavefront: 64 chunks of 16 bytes, ROWS rows of a unit's 128, the BN columns of the tile.  Chunk `lane` of
// request i of a wavefront that fetches REQUESTS of them lies in row first_row + i * ROWS of the unit, at column(lane, i) of
// the tile.
template <int BN>
struct KMajorRequests {
    static constexpr int CHUNKS = BN / 16, ROWS = 64 / CHUNKS;
    static HALO_HOST_DEVICE int first_row(int wave, int lane, int requests) { return wave * requests * ROWS + lane / CHUNKS; }
    static HALO_HOST_DEVICE int column(int lane, int i) {
        return 16 * ((lane % CHUNKS) ^ kmajor_swizzle<BN>(lane / CHUNKS) ^ kmajor_swizzle<BN>(i * ROWS));
    }
    // Columns that are fetched, from the tile's first one (n0): the matrix, in whole chunks.  Not the row pitch: of a matrix
    // that is a column slice of a wider one, the last row's pitch reaches past the end of the allocation.
    static HALO_HOST_DEVICE int64_t columns(int64_t N, int64_t n0) { return ((N + 15) & ~int64_t(15)) - n0; }
    // Offset from the tile's first column of the unit's first row.
    static HALO_HOST_DEVICE uint32_t offset(int row, int column, int64_t ldb, int64_t columns) {
        return column < columns ? (uint32_t)row * (uint32_t)ldb + (uint32_t)column : kOutside;
    }
};

}  // namespace halo
