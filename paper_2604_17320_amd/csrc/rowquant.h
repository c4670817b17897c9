// Row-quantizer pieces shared by the row kernels.  A row is owned by a GROUP of threads (one wave,
// or a whole 256-thread workgroup) and cached in registers as 16-byte chunks: chunk c belongs to
// thread c % GROUP of the group, as its (c / GROUP)-th chunk.
#pragma once
#include "common.h"
#include "internal.h"

#define ROW_THREADS 256
#define ROW_MAXCHUNK 16  // workgroup-per-row kernels: 16 chunks * 8 halves * 256 threads = 32768 columns
#define ROW_MAXCOLS 32768

// Where a quantized row goes: packed int4 (the public format, two codes per byte), the GEMM's A8 format --
// e4m3 bytes, every 8 codes as evens then odds, each row zero-padded to whole 128-channel groups, and behind the rows
// (if quota_a8_starts) what a sum of products with weights c + 8 starts from, [group][row] -- or, for at
// most 32 rows, packed int4 as the few-row GEMM's fragments: per 16 rows 1 KB per group, the 32 codes number q of row m's
// 128 at 16-byte piece 16 q + m % 16.  A null pointer drops the output.
struct RowOutPacked {
    static constexpr bool A8 = false, STARTS = false, MANY = true;       // MANY: launches of any number of rows
    uint32_t *q;
    static __device__ __forceinline__ int at(int c) { return c; }
};
struct RowOutFrag {
    static constexpr bool A8 = false, STARTS = false, MANY = false;
    uint32_t *q;
    static __device__ __forceinline__ int at(int c) { return (c >> 4) * 256 + (c >> 2 & 3) * 64 + (c & 3); }
};
struct RowOutA8 {
    static constexpr bool A8 = true, STARTS = false, MANY = false;       // (with_a8_out: less than quota_a8_starts)
    uint2 *q;
};
struct RowOutA8Starts {
    static constexpr bool A8 = true, STARTS = true, MANY = true;
    uint2 *q;
    int rows;            // of the launch
    float *starts;       // of this row
};
// run(the output of M rows in the A8 format)
template <typename RUN>
static inline int with_a8_out(void *qa8, int M, RUN run)
{
    if (quota_a8_starts(M)) return run(RowOutA8Starts{(uint2 *)qa8, M, nullptr});
    return run(RowOutA8{(uint2 *)qa8});
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
__host__ __device__ __forceinline__ RowOutA8 row_out(RowOutA8 o, size_t row, int nchunk)
{
    const int G = (nchunk + 15) >> 4;
    return RowOutA8{o.q + row * (G | 1) * 16};
}
__host__ __device__ __forceinline__ RowOutA8Starts row_out(RowOutA8Starts o, size_t row, int nchunk)
{
    const int G = (nchunk + 15) >> 4;
    return RowOutA8Starts{o.q + row * (G | 1) * 16, o.rows, reinterpret_cast<float *>(o.q + (size_t)o.rows * (G | 1) * 16) + row};
}

// final phase shared by the row kernels: quantize the cached row `v` with absmax `a`, store the
// codes, return this thread's share of the residual sum of squares.
template <bool WANT_RES, int GROUP, int NCH, typename OUT>
__device__ __forceinline__ double quantize_cached_row(const Pack16 *v, int nchunk, int idx, float a,
                                                      OUT out, float &s_out)
{
    float s = 1.0f, inv = 0.0f;
    if (a != 0.0f) { s = a / 7.0f; inv = 7.0f / a; }
    s_out = s;
    double rs = 0.0;
    const int nout = OUT::A8 ? (nchunk + 15) & ~15 : nchunk;
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        int c = idx + GROUP * r;
        if (c < nout) {
            const bool live = !OUT::A8 || c < nchunk;
            uint32_t word = 0;
            float unit[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = live ? (float)v[r].h[e] : 0.0f;
                const uint32_t cb = code_bits(f * inv);
                if (OUT::A8) {
                    unit[e] = code_unit(cb);
                } else {
                    word |= (cb & 0xFu) << (4 * e);
                }
                if (WANT_RES) {
                    float deq = code_float(cb) * s;
                    float rr = deq - f;
                    rs = __builtin_fma((double)rr, (double)rr, rs);     // product exact in fp64
                }
            }
            if constexpr (OUT::A8) {
                out.q[c] = units_to_e4m3(unit);
                if constexpr (OUT::STARTS) {         // the 16 lanes of a group add up in its last one
                    float u = ((unit[0] + unit[1]) + (unit[2] + unit[3])) + ((unit[4] + unit[5]) + (unit[6] + unit[7]));
                    u = row16_sum(u);
                    if ((c & 15) == 15) out.starts[(size_t)(c >> 4) * out.rows] = u * (-8.0f / 512.0f);
                }
            } else {
                if (out.q) out.q[OUT::at(c)] = word;
            }
        }
    }
    return rs;
}
