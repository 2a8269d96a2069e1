// edt_row.h -- occupancy bytes of a row to words of 32 bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace edt {

// Bits of 8 bytes (a then b): bit i set where byte i is nonzero.
__device__ inline uint32_t bytes8_bits(uint32_t a, uint32_t b) {
    // bit 7 of every byte: the byte is nonzero; the dot products weigh them
    // with 1, 2, 4, .. 128
    const uint32_t ta = ((((a & 0x7f7f7f7fu) + 0x7f7f7f7fu) | a) >> 7) & 0x01010101u;
    const uint32_t tb = ((((b & 0x7f7f7f7fu) + 0x7f7f7f7fu) | b) >> 7) & 0x01010101u;
    return __builtin_amdgcn_udot4(ta, 0x08040201u,
                                  __builtin_amdgcn_udot4(tb, 0x80402010u, 0u, false), false);
}
__device__ inline uint32_t bytes32_bits(const uint8_t* p) {
    uint32_t v[8];
    __builtin_memcpy(v, p, 32);                 // rows start at any byte
    return bytes8_bits(v[0], v[1]) | (bytes8_bits(v[2], v[3]) << 8) |
           (bytes8_bits(v[4], v[5]) << 16) | (bytes8_bits(v[6], v[7]) << 24);
}

// Occupancy word w (voxels 32 w .. 32 w + 31) of a row of nx voxels.
__device__ inline uint32_t row_word(const uint8_t* row, int nx, int w) {
    const int x0 = 32 * w;
    if (x0 + 32 <= nx) return bytes32_bits(row + x0);
    if (nx >= 32) return bytes32_bits(row + nx - 32) >> (x0 + 32 - nx);   // the row's last 32
    uint32_t m = 0u;
    for (int k = 0; k < nx; ++k) m |= (row[k] != 0 ? 1u : 0u) << k;
    return m;
}

}  // namespace edt
