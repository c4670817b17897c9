// Row-quantizer pieces shared by the row kernels.  A row is owned by a GROUP of threads (one wave,
// or a whole 256-thread workgroup) and cached in registers as 16-byte chunks: chunk c belongs to
// thread c % GROUP of the group, as its (c / GROUP)-th chunk.
#pragma once
#include "common.h"

#define ROW_THREADS 256
#define ROW_MAXCHUNK 16  // workgroup-per-row kernels: 16 chunks * 8 halves * 256 threads = 32768 columns
#define ROW_MAXCOLS 32768

// Where a quantized row goes: packed int4 (the public format, two codes per byte) or the GEMM's A8 format --
// e4m3 bytes, every 8 codes as evens then odds, each row zero-padded to whole 128-channel groups, plus
// the group sums times F8_CORR.  A null pointer drops the output.
struct RowOutPacked {
    static constexpr bool A8 = false;
    uint32_t *q;
};
struct RowOutA8 {
    static constexpr bool A8 = true;
    uint2 *q;
    float *corr;         // [ceil(G / 4)][M][4]: a wave's 64 chunks end in one 16-byte piece, and the GEMM's
    int M;               // lanes (neighbouring rows, same group) read pieces next to each other
};
__host__ __device__ __forceinline__ RowOutPacked row_out(RowOutPacked o, size_t row, int nchunk)
{
    return RowOutPacked{o.q ? o.q + row * nchunk : nullptr};
}
__host__ __device__ __forceinline__ RowOutA8 row_out(RowOutA8 o, size_t row, int nchunk)
{
    const int G = (nchunk + 15) >> 4;
    return RowOutA8{o.q + row * G * 16, o.corr + row * 4, o.M};
}

// final phase shared by the row kernels: quantize the cached row `v` with absmax `a`, store the
// codes, return this thread's share of the residual sum of squares.  GROUP is a multiple of 64, so
// the 16 chunks of a 128-channel group sit in 16 neighbouring lanes.
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
            float unit[8], sum = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = live ? (float)v[r].h[e] : 0.0f;
                const uint32_t cb = code_bits(f * inv);
                if (OUT::A8) {
                    unit[e] = __builtin_fmaf(__uint_as_float(cb), 1.0f / 512.0f, -ROW_MAGIC / 512.0f);  // code / 512, exact
                    sum += unit[e];
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
                int lo = __builtin_amdgcn_cvt_pk_fp8_f32(unit[0], unit[2], 0, false);
                lo = __builtin_amdgcn_cvt_pk_fp8_f32(unit[4], unit[6], lo, true);
                int hi = __builtin_amdgcn_cvt_pk_fp8_f32(unit[1], unit[3], 0, false);
                hi = __builtin_amdgcn_cvt_pk_fp8_f32(unit[5], unit[7], hi, true);
                out.q[c] = make_uint2((uint32_t)lo, (uint32_t)hi);
                // the group's 16 chunks are the 16 lanes of a DPP row: running sum, total in its last lane
#define STEP(ctrl) sum += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(sum), ctrl, 0xf, 0xf, true))
                STEP(0x111); STEP(0x112); STEP(0x114); STEP(0x118);
#undef STEP
                if ((c & 15) == 15) out.corr[(size_t)(c >> 6) * out.M * 4 + ((c >> 4) & 3)] = sum * (F8_CORR * 512.0f);
            } else {
                if (out.q) out.q[c] = word;
            }
        }
    }
    return rs;
}
