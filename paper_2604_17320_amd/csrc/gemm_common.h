// Pieces shared by the GEMM and attention kernels: int4 codes as e2m3 numbers, and the XCD-aware tile order.
#pragma once
#include "common.h"

// Sixteen codes as sixteen 6-bit e2m3 numbers in three dwords.  The multiples of 1/8 up to 15/8 are e2m3's linear range: the
// number of n / 8 has the bits 00nnnn, the sign on top.  Which of the sixteen a code becomes is free as long as weights and
// activations agree, and is chosen so that weights take few instructions: of the first eight codes each nibble stays at its bit,
// of the others each moves up by two, around the dword's end.  d0 takes the nibbles 0 3 6 of w0 and 1 4 and half of 7 of w1, d1
// 1 4 and half of 7 of w0 and the rest of 7 and 2 5 of w1, d2 the rest of 7 and 2 5 of w0 and 0 3 6 of w1.
constexpr uint32_t E6_STAY[3] = {0x0F00F00Fu, 0xF00F00F0u, 0x00F00F00u};     // of w0
constexpr uint32_t E6_MOVE[3] = {0xC03C03C0u, 0x03C03C03u, 0x3C03C03Cu};     // of w1, two bits up
constexpr uint32_t E6_FLIP[3] = {0x08208208u, 0x82082082u, 0x20820820u};     // the top bits of the codes: c -> c + 8

// Weights, as c + 8.  Seven instructions for 16 codes (eight, with the first codes moved too: a layer of 11264 rows 1349 -> 1336 us, of
// 640 160.9 -> 159.4).  `flip` holds E6_FLIP in vector registers: an instruction reads one
// constant from the scalar ones.
__device__ __forceinline__ void weights_e2m3(uint32_t w0, uint32_t w1, const uint32_t (&flip)[3], int &d0, int &d1, int &d2)
{
    const uint32_t up = __builtin_amdgcn_alignbit(w1, w1, 30);
    auto pick = [&](int i) {                                                 // (w0 & STAY ^ FLIP) ^ (up & MOVE)
        return (int)__builtin_amdgcn_bitop3_b32(__builtin_amdgcn_bitop3_b32(w0, E6_STAY[i], flip[i], 0x6A), up, E6_MOVE[i], 0x78);
    };
    d0 = pick(0);
    d1 = pick(1);
    d2 = pick(2);
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
    const uint32_t mag = (e.x & low) | (e.y << 4 & ~low), sign = (e.x >> 4 & 0x08080808u) | (e.y & 0x80808080u);
    // A zero has no sign: a product's bits would change with it for nothing, and the chip lowers its clock for that (8 x 640 rows of the 13B
    // shape, whole layers: 1.5 % longer with zeros of both signs).
    return {mag, sign & (((mag & 0x77777777u) + 0x77777777u) | mag)};
}
__device__ __forceinline__ int sum_of(const Codes8 &c)
{
    const uint32_t negative = c.sign | (c.sign - (c.sign >> 3));             // whole nibbles
    return (int)__builtin_amdgcn_udot8(c.mag, 0x11111111u, 0, false) -
           2 * (int)__builtin_amdgcn_udot8(c.mag & negative, 0x11111111u, 0, false);
}
// What the first (second) eight codes of sixteen give to d0, d1 and d2.  Masks and shifts of a lane that always has the one or the
// other can be made once.
struct E6Masks { uint32_t mag[3], sign[3]; int mag_right, sign_right; };
__device__ __forceinline__ E6Masks e2m3_masks(bool second)
{
    E6Masks k;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t stay = E6_STAY[i] & 0x88888888u, top = E6_FLIP[i] & ~stay;        // top bits of the nibbles that stay, that move
        const int before = (i + 2) % 3;                  // (a sign lies two bits above its nibble: it may be the next dword's)
        const uint32_t stay0 = E6_STAY[before] & 0x88888888u, top0 = E6_FLIP[before] & ~stay0;
        k.mag[i] = second ? E6_MOVE[i] : E6_STAY[i];
        k.sign[i] = second ? (top << 2 | top0 >> 30) : (stay << 2 | stay0 >> 30);
    }
    k.mag_right = second ? 30 : 0;
    k.sign_right = second ? 28 : 30;
    return k;
}
__device__ __forceinline__ void codes_e2m3(const Codes8 &c, const E6Masks &k, uint32_t (&d)[3])
{
    const uint32_t m = __builtin_amdgcn_alignbit(c.mag, c.mag, k.mag_right), s = __builtin_amdgcn_alignbit(c.sign, c.sign, k.sign_right);
#pragma unroll
    for (int i = 0; i < 3; ++i) d[i] = (m & k.mag[i]) | (s & k.sign[i]);
}
// 32 packed int4 codes (one 16-byte piece): six dwords
__device__ __forceinline__ void codes_e2m3(const i32x4 &v, uint32_t (&d)[6])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t first[3], second[3];
        codes_e2m3(codes_of_nibbles((uint32_t)v[2 * i]), e2m3_masks(false), first);
        codes_e2m3(codes_of_nibbles((uint32_t)v[2 * i + 1]), e2m3_masks(true), second);
#pragma unroll
        for (int j = 0; j < 3; ++j) d[3 * i + j] = first[j] | second[j];
    }
}

// Tile order inside an XCD's range: bands of 8 row tiles, column by column, so that the 64 or so workgroups
// an XCD runs at a time cover about 8 x 8 tiles and share their operands in its L2 (row tiles first
// would give every workgroup its own activations: at 11264 rows that cost 2x in traffic beyond L2).
__device__ __forceinline__ void tile_of(int tile, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const unsigned wide = 8u * (unsigned)tiles_n, band = (unsigned)tile / wide, first = 8 * band, rows = min(8u, (unsigned)tiles_m - first);
    const unsigned i = (unsigned)tile - band * wide;
    tn = (int)(i / rows);
    tm = (int)(first + i - (unsigned)tn * rows);
}
