// Shared device helpers for the gfx950 kernels of libquota (wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include "../../include/quota.h"
#include "profile.h"

#define QUOTA_WAVE 64

// launch-error check used by every host entry point after it enqueues kernels
#define QUOTA_RETURN_IF_LAUNCH_FAILED()                    \
    do {                                                   \
        if (hipGetLastError() != hipSuccess) return QUOTA_ERR_HIP; \
    } while (0)

typedef _Float16 f16;
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Vectors at addresses aligned as their elements are: the chip takes them with the same 16-byte instructions.
// For tensors whose caller promises no more than that.
typedef f16x8 f16x8_at2 __attribute__((aligned(2)));
typedef f32x4 f32x4_at4 __attribute__((aligned(4)));
typedef uint32_t u32_at2 __attribute__((aligned(2), may_alias));
__device__ __forceinline__ uint4 load16_at2(const f16 *p)
{
    return __builtin_bit_cast(uint4, *reinterpret_cast<const f16x8_at2 *>(p));
}
__device__ __forceinline__ void store16_at2(f16 *p, const uint4 &v)
{
    *reinterpret_cast<f16x8_at2 *>(p) = __builtin_bit_cast(f16x8, v);
}

union Pack16 {           // 16 bytes seen as halves, dwords or one vector load
    uint4 u;
    f16 h[8];
    uint32_t w[4];
};

// Wave-wide reductions with DPP moves (no LDS crossbar): an inclusive scan -- shifts by 1, 2, 4, 8
// inside each row of 16 lanes, then lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into
// rows 2 and 3 -- leaves the result of all 64 lanes in lane 63, which is read back as a scalar.
// Lanes without a source combine with the operation's identity.
#define QUOTA_DPP_STEPS(STEP) \
    STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf) STEP(0x142, 0xa) STEP(0x143, 0xc)

__device__ __forceinline__ float wave_max(float v)
{
#define STEP(ctrl, rows)                                                                              \
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, \
                                                            rows, 0xf, false)));
    QUOTA_DPP_STEPS(STEP)
#undef STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// ... of values that are not negative (no NaN): their bits order as integers do, which leaves one instruction a step where the
// float maximum takes four (it first makes a quiet NaN of a signalling one that might have come along)
__device__ __forceinline__ float wave_absmax(float v)
{
    uint32_t u = __float_as_uint(v);
#define STEP(ctrl, rows) u = max(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, ctrl, rows, 0xf, false));
    QUOTA_DPP_STEPS(STEP)
#undef STEP
    return __int_as_float(__builtin_amdgcn_readlane((int)u, 63));
}
__device__ __forceinline__ double wave_sum(double v)
{
#define STEP(ctrl, rows)                                                                       \
    {                                                                                          \
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, rows, 0xf, false); \
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, rows, 0xf, false); \
        v += __hiloint2double(hi, lo);                                                         \
    }
    QUOTA_DPP_STEPS(STEP)
#undef STEP
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}
__device__ __forceinline__ float wave_sum(float v)
{
#define STEP(ctrl, rows) \
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xf, false));
    QUOTA_DPP_STEPS(STEP)
#undef STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// sum or maximum over each row of 16 lanes, in all of them
__device__ __forceinline__ double row16_all(double v)
{
#define STEP(ctrl)                                                                                          \
    v += __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true),                \
                          __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true));
    STEP(0xB1) STEP(0x4E) STEP(0x141) STEP(0x140)          // from lane 1 and 2 over, from the other half's mirror, the row's
#undef STEP
    return v;
}
__device__ __forceinline__ uint32_t row16_all(uint32_t v)
{
#define STEP(ctrl) v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, ctrl, 0xf, 0xf, true));
    STEP(0xB1) STEP(0x4E) STEP(0x141) STEP(0x140)
#undef STEP
    return v;
}

// sum over each row of 16 lanes, in its last lane
__device__ __forceinline__ float row16_sum(float v)
{
#define STEP(ctrl) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false));
    STEP(0x111) STEP(0x112) STEP(0x114) STEP(0x118)
#undef STEP
    return v;
}

// The fp32 number nearest to 1 / sqrt(x).  A division by a square root in doubles is a chain of some forty instructions in front of
// everything a row's normalisation does; the estimate y is good to 2^-23, so that e = 1 - x y^2 is below 2^-22, and three terms of
// y (1 - e)^(-1/2) = y (1 + e / 2 + 3 e^2 / 8 + 5 e^3 / 16 + ...) leave an error of 2^-67.7 and the last roundings'.  Over 4 million x from 1e-12 to 4e9 and estimates
// off by up to 2^-22 the result is 1.24 x 2^-53 off at most, the division by the root 1.49, and both round to the nearest fp32 number every time.
__device__ __forceinline__ float inv_sqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x), e = __builtin_fma(-x * y, y, 1.0);
    const double r = __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
    return (float)(x > 0.0 && x < INFINITY ? r : y);             // 0, infinity and NaN: e is none
}

// Sum and / or maximum (of floats that are not negative) over waves `first` to `first` + NW - 1 of a workgroup, NW a power of two up to
// 8, in all their threads.  Every 16 lanes leave theirs in LDS; a lane reads two of the 4 NW and adds them up with its neighbours'.
// (Every lane reading all of them takes the LDS of a CU some 400 clocks for 8 waves, this 100.)  A barrier of the
// whole workgroup in between.  FRESH: nothing read `sums` or `maxima` (4 each per wave of the workgroup, as wanted) in this workgroup before.
template <bool MAX, bool SUM, bool FRESH>
__device__ __forceinline__ void waves_max_sum(float &mx, double &sum, double *sums, uint32_t *maxima, int wave, int first, int nw)
{
    const int lane = threadIdx.x & 63, put = 4 * wave + (lane >> 4), get = 4 * first + 2 * (lane & (2 * nw - 1));
    const bool reads = (lane & 15) < 2 * nw;                  // (the others add nothing)
    uint32_t m = 0;
    if (MAX) m = row16_all(__float_as_uint(mx));
    if (SUM) sum = row16_all(sum);
    if (!FRESH) __syncthreads();
    if ((lane & 15) == 0) {
        if (MAX) maxima[put] = m;
        if (SUM) sums[put] = sum;
    }
    __syncthreads();
    uint2 m2 = make_uint2(0, 0);
    double2 s2 = make_double2(0.0, 0.0);
    if (MAX) m2 = *reinterpret_cast<const uint2 *>(maxima + get);
    if (SUM) s2 = *reinterpret_cast<const double2 *>(sums + get);
    if (MAX) mx = __uint_as_float(row16_all(reads ? max(m2.x, m2.y) : 0u));
    if (SUM) sum = row16_all(reads ? s2.x + s2.y : 0.0);
}
// ... over all NW of them; `sm`, aligned to 16 bytes, needs 6 * NW doubles of LDS.
template <int NW, bool MAX, bool SUM, bool FRESH = false>
__device__ __forceinline__ void block_max_sum(float &mx, double &sum, double *sm)
{
    waves_max_sum<MAX, SUM, FRESH>(mx, sum, sm, reinterpret_cast<uint32_t *>(sm + 4 * NW), (int)(threadIdx.x >> 6), 0, NW);
}

// Consecutive workgroups go round-robin over the 8 XCDs, each with its own L2: this gives each XCD a contiguous range
// of ids.
__device__ __forceinline__ int xcd_remap(int pid, int total)
{
    int x = pid & 7, idx = pid >> 3;
    int per = total >> 3, rem = total & 7;
    return x * per + (x < rem ? x : rem) + idx;
}

// fp32 -> fp16 with the fp32 value materialised first.  Without the barrier
// the compiler may fold "multiply/add, then convert" into one mixed-precision
// instruction that rounds the exact result straight to fp16; the two-step
// rounding written here is what the rest of the pipeline is defined with.
__device__ __forceinline__ f16 to_f16(float v)
{
    asm volatile("" : "+v"(v));
    return (f16)v;
}

// silu(gate) * up, silu(g) = g / (1 + e^-g) with the hardware exp2 and reciprocal (a few fp32 ulp, far inside the fp16
// rounding that follows)
__device__ __forceinline__ f16 silu_mul(float gate, float up)
{
    const float s = gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate));
    return to_f16(s * up);
}

// int4 code from a rounded fp32 value: clamp to [-8, 7]
__device__ __forceinline__ int code_from(float r)
{
    r = fminf(fmaxf(r, -8.0f), 7.0f);
    return (int)r;
}

// s = a / 7 and inv = 7 / a of a row's absmax, an fp16 number; 1 and 0 for a = 0.  The same bits as the divisions', which take
// some ten dependent instructions each: the quotient by the reciprocal, corrected once by its exact remainder, is the
// nearest number for every finite fp16 a, whichever reciprocal within one unit in the last place the estimate is.
__device__ __forceinline__ void sevenths(float a, float &s, float &inv)
{
    constexpr float SEVENTH = 1.0f / 7.0f;
    const float qs = a * SEVENTH, y0 = __builtin_amdgcn_rcpf(a);
    const float y = __builtin_fmaf(__builtin_fmaf(-a, y0, 1.0f), y0, y0), qi = 7.0f * y;
    s = __builtin_fmaf(__builtin_fmaf(-7.0f, qs, a), SEVENTH, qs);
    inv = __builtin_fmaf(__builtin_fmaf(-a, qi, 7.0f), y, qi);
    if (!(a < INFINITY)) { s = a; inv = 0.0f; }
    if (a == 0.0f) { s = 1.0f; inv = 0.0f; }
}

// The int4 code of a scaled value t = x * (7 / absmax), without a round / convert / mask chain:
// clamp to [-8, 7] first (the bounds are integers, so clamping commutes with rounding to integer),
// then add 1.5 * 2^23 -- in that binade one unit in the last place is 1, so the fp32 add itself
// rounds to the nearest integer, ties to even, and the low mantissa bits of the sum hold the code in
// two's complement.  code_bits(t) & 0xF is the packed nibble; code_float(bits) the code as a float.
#define ROW_MAGIC 12582912.0f
__device__ __forceinline__ uint32_t code_bits(float t)
{
    t = fminf(fmaxf(t, -8.0f), 7.0f);          // NaN -> -8, as in code_from
    return __float_as_uint(t + ROW_MAGIC);
}
// Units of the GEMM operands: code / 8 is an e2m3 number for every int4 code, so a group's accumulator counts in 2^-6 (see
// gemm.hip); as e4m3 numbers (rows16.hip), code / 512, it counts in 2^-18.
#define F6_UNIT 64.0f
#define F8_UNIT 262144.0f
// 8 such units as e4m3 bytes, evens then odds
__device__ __forceinline__ uint2 units_to_e4m3(const float unit[8])
{
    int lo = __builtin_amdgcn_cvt_pk_fp8_f32(unit[0], unit[2], 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(unit[4], unit[6], lo, true);
    int hi = __builtin_amdgcn_cvt_pk_fp8_f32(unit[1], unit[3], 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(unit[5], unit[7], hi, true);
    return make_uint2((uint32_t)lo, (uint32_t)hi);
}
__device__ __forceinline__ float code_float(uint32_t bits) { return __uint_as_float(bits) - ROW_MAGIC; }

