// Pieces shared by the GEMM and attention kernels: int4 codes as e4m3 bytes, and the XCD-aware tile order.
#pragma once
#include "common.h"

// 32 packed int4 codes (one 16-byte piece) as signed e4m3 bytes in the A8 order -- every 8 codes as evens
// then odds.  With u = code & 15 and b its sign bit the e4m3 byte is u for b = 0 and
// 0x90 - u = (u ^ 15) + 0x81 for b = 1, IN UNITS OF 1/512 (the linear range of e4m3), so that no
// table is needed; v_xad_u32 does the last step.
__device__ __forceinline__ uint32_t nibbles_to_e4m3(uint32_t u)
{
    const uint32_t t = u & 0x08080808u, b = t >> 3;
    return (u ^ (t | (t - b))) + ((t << 4) | b);
}
__device__ __forceinline__ void codes_to_e4m3(const uint4 &v, uint4 &e0, uint4 &e1)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t e[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        e[2 * i] = nibbles_to_e4m3(w[i] & 0x0F0F0F0Fu);
        e[2 * i + 1] = nibbles_to_e4m3((w[i] >> 4) & 0x0F0F0F0Fu);
    }
    e0 = make_uint4(e[0], e[1], e[2], e[3]);
    e1 = make_uint4(e[4], e[5], e[6], e[7]);
}

// Tile order inside an XCD's range: bands of 8 row tiles, column by column, so that the 64 or so workgroups
// an XCD runs at a time cover about 8 x 8 tiles and share their operands in its L2 (row tiles first
// would give every workgroup its own activations: at 11264 rows that cost 2x in traffic beyond L2).
__device__ __forceinline__ void tile_of(int tile, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const int band = tile / (8 * tiles_n), first = 8 * band, rows = min(8, tiles_m - first);
    const int i = tile - band * 8 * tiles_n;
    tm = first + i % rows;
    tn = i / rows;
}
