// Row-quantizer pieces shared by the row kernels.  A row is owned by a GROUP of threads (one wave,
// or a whole workgroup of 256 or 512 threads) and cached in registers as 16-byte chunks: chunk c belongs to
// thread c % GROUP of the group, as its (c / GROUP)-th chunk.
#pragma once
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "gemm_common.h"

#define ROW_THREADS 256
#define ROW_MAXCHUNK 16  // workgroup-per-row kernels: 16 chunks * 8 halves * 256 threads = 32768 columns, as 8 chunks of 512 threads
#define ROW_MAXCOLS 32768

// Where a quantized row goes: packed int4 (the public format, two codes per byte), the GEMM's A6 format -- e2m3 numbers,
// zero-padded to whole 128-channel groups; for every four rows and group 384 bytes, of row r from 64 r on the first four of the six
// dwords of each 32 channels, from 256 + 32 r on the others -- and behind the rows
// (if quota_a6_starts) what a sum of products with weights c + 8 starts from, [group][row] -- or, for at
// most 32 rows, packed int4 as the few-row GEMM's fragments: per 16 rows 1 KB per group, the 32 codes number q of row m's
// 128 at 16-byte piece 16 q + m % 16.  A null pointer drops the output.
struct RowOutPacked {
    static constexpr bool A6 = false, STARTS = false, MANY = true;       // MANY: launches of any number of rows
    uint32_t *q;
    static __device__ __forceinline__ int at(int c) { return c; }
};
struct RowOutFrag {
    static constexpr bool A6 = false, STARTS = false, MANY = false;
    uint32_t *q;
    static __device__ __forceinline__ int at(int c) { return (c >> 4) * 256 + (c >> 2 & 3) * 64 + (c & 3); }
};
struct RowOutA6 {
    static constexpr bool A6 = true, STARTS = false, MANY = false;       // (with_a6_out: less than quota_a6_starts)
    uint32_t *q;
};
struct RowOutA6Starts {
    static constexpr bool A6 = true, STARTS = true, MANY = true;
    uint32_t *q;
    int rows;            // of the launch
    float *starts;       // of this row
};
// run(the output of M rows in the A6 format)
template <typename RUN>
static inline int with_a6_out(void *qa6, int M, RUN run)
{
    if (quota_a6_starts(M)) return run(RowOutA6Starts{(uint32_t *)qa6, M, nullptr});
    return run(RowOutA6{(uint32_t *)qa6});
}
// The row (or rows) that workgroup `wg` takes: with start values, 4 bytes per row and group, neighbouring rows belong on one XCD, whose L2
// puts them together (5808 rows and 11008 columns: 0.4 % of a layer's time).
template <typename OUT>
__device__ __forceinline__ int row_wg(int wg, int wgs)
{
    if constexpr (OUT::STARTS) return xcd_remap(wg, wgs);
    return wg;
}
__host__ __device__ __forceinline__ RowOutPacked row_out(RowOutPacked o, size_t row, int nchunk)
{
    return RowOutPacked{o.q ? o.q + row * nchunk : nullptr};
}
__host__ __device__ __forceinline__ RowOutFrag row_out(RowOutFrag o, size_t row, int nchunk)
{
    return RowOutFrag{o.q + (row >> 4) * ((nchunk + 15) >> 4) * 256 + 4 * (row & 15)};
}
// (bytes of four rows fit 32 bits)
__host__ __device__ __forceinline__ uint32_t *a6_row(uint32_t *q, size_t row, int G)
{
    return q + ((size_t)(unsigned)(row >> 2) * ((unsigned)quota_a6_groups(G) * 96u) + ((unsigned)row & 3) * 16);
}
__host__ __device__ __forceinline__ RowOutA6 row_out(RowOutA6 o, size_t row, int nchunk)
{
    return RowOutA6{a6_row(o.q, row, (nchunk + 15) >> 4)};
}
__host__ __device__ __forceinline__ RowOutA6Starts row_out(RowOutA6Starts o, size_t row, int nchunk)
{
    const int G = (nchunk + 15) >> 4;
    return RowOutA6Starts{a6_row(o.q, row, G), o.rows,
                          reinterpret_cast<float *>(o.q + (((size_t)o.rows + 3) >> 2) * quota_a6_groups(G) * 96) + row};
}
// Stores chunks (8 channels) of a row in the A6 format, chunk c by a thread whose chunks are all idx modulo 64; four
// neighbouring lanes hold the chunks of 32 channels.  A pair's lanes put their shares of d0, d1 and d2 together; its first stores d0, its
// second d1 and d2.  Masks and the place inside a group are the thread's own, made once: by kernels of a workgroup per row while they
// wait for it, by kernels of a wave per row when the sums are done (their registers are what limits the rows in flight: early, 11264
// rows of 4096 columns took 8 more, four waves a SIMD instead of five).
typedef uint32_t u32x2_at4 __attribute__((ext_vector_type(2), aligned(4), may_alias));
struct E6Store {
    E6Masks k;
    unsigned at;                         // bytes from the row's first dword to this thread's place in a group
    __device__ __forceinline__ void make(int idx, int row)
    {
        k = e2m3_masks(idx & 1);
        const unsigned quarter = idx >> 2 & 3, main = quarter * 16, tail = 256 - 32 * (row & 3) + quarter * 8;
        at = idx & 1 ? (idx & 2 ? tail : main + 4) : main + (idx & 2 ? 12 : 0);
#pragma unroll
        for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(k.mag[i]), "+v"(k.sign[i]));  // (else they are selected anew for every chunk)
    }
    __device__ __forceinline__ void operator()(uint32_t *row_q, int c, const Codes8 &codes) const
    {
        uint32_t d[3];
        codes_e2m3(codes, k, d);
#pragma unroll
        for (int i = 0; i < 3; ++i) d[i] |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d[i], 0xB1, 0xf, 0xf, false);    // quad lanes 1 0 3 2
        // (one lane of four storing all 16 bytes of the first part, another the second, takes longer: 5808 x 11008 42.7 us, 40.1 so)
        char *to = (char *)row_q + (at + (unsigned)(c >> 4) * 384u);
        if (c & 1) *reinterpret_cast<u32x2_at4 *>(to) = u32x2_at4{d[1], d[2]};
        else *reinterpret_cast<uint32_t *>(to) = d[0];
    }
};
// What the final phase below is handed for a row of the format OUT: an E6Store, or nothing
struct NoStore {
    __device__ __forceinline__ void make(int, int) {}
};
template <typename OUT>
using RowStore = std::conditional_t<OUT::A6, E6Store, NoStore>;

// final phase shared by the row kernels: quantize the cached row `v` with absmax `a`, store the
// codes, return this thread's share of the residual sum of squares.
template <bool WANT_RES, int GROUP, int NCH, typename OUT>
__device__ __forceinline__ double quantize_cached_row(const Pack16 *v, int nchunk, int idx, float a,
                                                      OUT out, const RowStore<OUT> &store, float &s_out)
{
    float s, inv;
    sevenths(a, s, inv);
    s_out = s;
    static_assert(!(OUT::A6 && WANT_RES), "(chunks past the row repeat one)");
    double rs = 0.0;
    const int nout = OUT::A6 ? (nchunk + 15) & ~15 : nchunk;
    const float inv_unit = inv * (1.0f / 512.0f);                // (exact)
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        int c = idx + GROUP * r;
        if (c < nout) {
            if constexpr (OUT::A6) {
                // The conversion to e4m3 rounds x * inv / 512 to the nearest multiple of 1/512, ties to even, as code_bits rounds
                // x * inv to an integer.  No bound above: |x| <= a, and 7.0000005 rounds to 7; NaN -> -8, as there.  Two instructions an
                // element where code_bits and the way back to a number took five (with the masks ahead of the row and
                // the maximum by integers, us: 42 x 512 2.68 -> 2.47, RMSNorm 3.15 -> 2.99, 640 x 11008 6.83 -> 6.33; stacks of 16 layers of 512
                // channels, 42 to 320 rows 2 % less, decode steps of 33 to 64 rows 4 %).
                float unit[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) unit[e] = fmaxf((float)v[r].h[e] * inv_unit, -8.0f / 512.0f);
                uint2 b = units_to_e4m3(unit);
                b = c < nchunk ? b : make_uint2(0, 0);           // (chunks that fill a group up)
                const Codes8 codes = codes_of_e4m3(b);
                store(out.q, c, codes);
                if constexpr (OUT::STARTS) {                     // the 16 lanes of a group add up in its last one
                    const float u = row16_sum((float)sum_of(codes));
                    if ((c & 15) == 15) out.starts[(size_t)(c >> 4) * out.rows] = u * (-8.0f / 64.0f);       // -8 / 8 times the sum of codes / 8
                }
            } else {
                uint32_t word = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float f = (float)v[r].h[e];
                    const uint32_t cb = code_bits(f * inv);
                    word |= (cb & 0xFu) << (4 * e);
                    if (WANT_RES) {
                        float deq = code_float(cb) * s;
                        float rr = deq - f;
                        rs = __builtin_fma((double)rr, (double)rr, rs);     // product exact in fp64
                    }
                }
                if (out.q) out.q[OUT::at(c)] = word;
            }
        }
    }
    return rs;
}
