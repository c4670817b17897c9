// Pieces shared by the GEMM and attention kernels: int4 codes as e2m3 numbers, and the XCD-aware tile order.
#pragma once
#include "common.h"

// Sixteen codes as sixteen 6-bit e2m3 numbers in three dwords.  The multiples of 1/8 up to 15/8 are e2m3's linear range: the
// number of n / 8 has the bits 00nnnn, the sign on top.  Which of the sixteen a code becomes is free as long as weights and
// activations agree, and is chosen so that weights take few instructions: a nibble stays at its bit or moves up by two.  Of
// w0 (codes 0 to 7) and w1 (8 to 15), d0 takes 0 1 3 4 6 and the low half of 7, d1 the rest of 7 and 9 10 12 13 15,
// d2 2 5 8 11 14.
constexpr uint32_t E6_STAY[3] = {0x0F00F00Fu, 0xF00F00F0u, 0x00F00F00u};     // of w0, w1, w0
constexpr uint32_t E6_MOVE[3] = {0xC03C03C0u, 0x03C03C03u, 0x3C03C03Cu};     // of w0, w1 (and w0), w1, two bits up
constexpr uint32_t E6_FLIP[3] = {0x08208208u, 0x82082082u, 0x20820820u};     // the top bits of the codes: c -> c + 8

// Weights, as c + 8.  Eight instructions for 16 codes.  `flip` holds E6_FLIP in vector registers: an instruction reads one
// constant from the scalar ones.
__device__ __forceinline__ void weights_e2m3(uint32_t w0, uint32_t w1, const uint32_t (&flip)[3], int &d0, int &d1, int &d2)
{
    const uint32_t up0 = w0 << 2, up1 = __builtin_amdgcn_alignbit(w1, w0, 30);
    auto pick = [&](uint32_t stay, uint32_t move, int i) {                   // (stay & STAY ^ FLIP) ^ (move & MOVE)
        return (int)__builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(stay, E6_STAY[i], flip[i], 0x6A), move, E6_MOVE[i], 0x78);
    };
    d0 = pick(w0, up0, 0);
    d1 = pick(w1, up1, 1);
    d2 = pick(w0, up1, 2);
}
__device__ __forceinline__ void e2m3_flips(uint32_t (&flip)[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        flip[i] = E6_FLIP[i];
        asm("" : "+v"(flip[i]));
    }
}
// 32 packed weights as an operand
__device__ __forceinline__ void weights_e2m3(const uint4 &w, const uint32_t (&flip)[3], i32x8 &f)
{
    int d[6];
    weights_e2m3(w.x, w.y, flip, d[0], d[1], d[2]);
    weights_e2m3(w.z, w.w, flip, d[3], d[4], d[5]);
    f = i32x8{d[0], d[1], d[2], d[3], d[4], d[5], 0, 0};
}

// Activations, as signed numbers: eight codes as magnitudes (nibbles) and signs (their top bits).
struct Codes8 { uint32_t mag, sign; };
__device__ __forceinline__ Codes8 codes_of_nibbles(uint32_t w)               // two's complement
{
    const uint32_t s = w & 0x88888888u, one = s >> 3;
    return {((w ^ (s - one)) & 0x77777777u) + one, s};
}
__device__ __forceinline__ Codes8 codes_of_e4m3(const uint2 &e)              // units_to_e4m3: sign and magnitude in a byte
{
    const uint32_t low = 0x0F0F0F0Fu;
    return {(e.x & low) | (e.y << 4 & ~low), (e.x >> 4 & 0x08080808u) | (e.y & 0x80808080u)};
}
// What the first (second) eight codes of sixteen give to d0, d1, d2: own = to d0 (d1), d2, and of the first, to d1.  The masks of
// a lane that always has the one or the other can be made once.
struct E6Masks { uint32_t own[4], d2[5]; };
__device__ __forceinline__ E6Masks e2m3_masks(bool second)
{
    return {{second ? E6_STAY[1] : E6_STAY[0], second ? E6_MOVE[1] & ~3u : E6_MOVE[0], second ? 0x00200200u : 0x20020020u,
             second ? 0x08008000u : 0x00800800u},
            {second ? 0u : E6_STAY[2], second ? E6_MOVE[2] : 0u, second ? 0u : 0x02002000u, second ? 0x80080080u : 0u, second ? 2u : 0u}};
}
__device__ __forceinline__ void codes_e2m3(const Codes8 &c, const E6Masks &k, uint32_t &own, uint32_t &d2, uint32_t &d1)
{
    const uint32_t m = c.mag, m2 = m << 2, s2 = c.sign << 2, s4 = c.sign << 4;
    own = (m & k.own[0]) | (m2 & k.own[1]) | (s2 & k.own[2]) | (s4 & k.own[3]);
    d2 = (m & k.d2[0]) | (m2 & k.d2[1]) | (s2 & k.d2[2]) | (s4 & k.d2[3]) | (c.sign >> 30 & k.d2[4]);
    d1 = (m >> 30) | (c.sign >> 28 & 8u);
}
// 32 packed int4 codes (one 16-byte piece): six dwords
__device__ __forceinline__ void codes_e2m3(const i32x4 &v, uint32_t (&d)[6])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t o0, o1, a2, b2, a1, b1;
        codes_e2m3(codes_of_nibbles((uint32_t)v[2 * i]), e2m3_masks(false), o0, a2, a1);
        codes_e2m3(codes_of_nibbles((uint32_t)v[2 * i + 1]), e2m3_masks(true), o1, b2, b1);
        d[3 * i] = o0;
        d[3 * i + 1] = o1 | a1;
        d[3 * i + 2] = a2 | b2;
    }
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
