// RoPE and the 4-bit K/V group quantizer on one 8-channel chunk, shared by the stand-alone
// RoPE/KV kernel and the fused epilogue of the QKV GEMM (both must round identically).
#pragma once
#include "common.h"

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// (float)h * f, rounded once, as one instruction that reads the half as it is: a multiply-add with -0, which changes
// nothing, in a register, or the compiler makes it a conversion and a product.
struct MixMul {
    float minus0 = -0.0f;
    __device__ __forceinline__ MixMul() { asm volatile("" : "+v"(minus0)); }
    __device__ __forceinline__ float operator()(f16 h, float f) const { return __builtin_fmaf((float)h, f, minus0); }
};
// two fp32 values rounded to fp16 (see to_f16)
__device__ __forceinline__ f16x2 to_f16x2(float a, float b)
{
    asm volatile("" : "+v"(a), "+v"(b));
    return __builtin_convertvector(f32x2{a, b}, f16x2);
}

// Maximum over the 8 lanes [lane & ~7, +8): across pairs, pairs of pairs, and the two quads, which are mirrored
__device__ __forceinline__ float lanes8_max(float a)
{
#define STEP(ctrl) a = fmaxf(a, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), ctrl, 0xf, 0xf, true)));
    STEP(0xB1) STEP(0x4E) STEP(0x141)
#undef STEP
    return a;
}

// Quantize this lane's 8 channels; the 8 lanes [lane & ~7, +8) form one 64-channel group and
// must all call this together.  Returns packed codes; *sh_out = fp16 group scale; xhat
// (optional) = fp16(code * scale), the value attention sees.
// Instructions count here: with IEEE divisions, shuffles through LDS, a shift per code and its index arithmetic the epilogue of
// a 128 x 256 tile of the QKV projection had 4525 vector instructions a thread, 70 % of its main loop's at 4096 channels; it has 2580
// (16 x 704 tokens of the 7B shape, whole layer: 1565 -> 1475 us).  The scale a / 7 has only to be right in fp16, where a * (1 / 7)
// gives the same for every fp16 a; one step of Newton's method makes the reciprocal of an fp16 number the correctly rounded
// one (both checked over all of them); four codes are packed by multiply-adds; code * scale is exact before its rounding
// to fp16.
__device__ __forceinline__ uint32_t kv_quant8(const Pack16 &x, f16 *sh_out, Pack16 *xhat, const MixMul &mul = MixMul())
{
    float a = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf((float)x.h[e]));
    a = lanes8_max(a);
    f16 sh = to_f16(a * (1.0f / 7.0f));
    if ((float)sh == 0.0f) sh = (f16)1.0f;
    const float s = (float)sh, r0 = __builtin_amdgcn_rcpf(s);
    const float r = __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-s, r0, 1.0f), r0, r0), s, 1.0f);       // (s = inf: 0)
    float c[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) c[e] = code_float(code_bits(mul(x.h[e], r)));
    uint32_t half[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {       // c + 8 of four codes, in the low mantissa bits
        float p = c[4 * i] + (ROW_MAGIC + 8.0f * (1 + 16 + 256 + 4096));
        p = __builtin_fmaf(c[4 * i + 1], 16.0f, p);
        p = __builtin_fmaf(c[4 * i + 2], 256.0f, p);
        p = __builtin_fmaf(c[4 * i + 3], 4096.0f, p);
        half[i] = __float_as_uint(p);
    }
    if (xhat) {
        f16x2 *o = reinterpret_cast<f16x2 *>(xhat->h);
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = __builtin_convertvector(f32x2{c[2 * i], c[2 * i + 1]}, f16x2) * f16x2{sh, sh};
    }
    *sh_out = sh;
    return __builtin_amdgcn_perm(half[1], half[0], 0x05040100u) ^ 0x88888888u;
}

// Rotate-half RoPE of one chunk: x holds channels [8c, 8c+8) of a head, xp the partner chunk
// half a head away, cs / sn the angle table entries of these 8 pair indices; `second` says
// whether x lies in the second half of the head.  fp32 products, one add, rounded to fp16.
__device__ __forceinline__ void rope8(const Pack16 &x, const Pack16 &xp, const float cs[8],
                                      const float sn[8], bool second, Pack16 &out, const MixMul &mul = MixMul())
{
    const uint32_t flip = second ? 0u : 0x80008000u;
    Pack16 xs;
#pragma unroll
    for (int i = 0; i < 4; ++i) xs.w[i] = xp.w[i] ^ flip;
    f16x2 *o = reinterpret_cast<f16x2 *>(out.h);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
            v[e] = mul(x.h[2 * i + e], cs[2 * i + e]) + mul(xs.h[2 * i + e], sn[2 * i + e]);
        o[i] = to_f16x2(v[0], v[1]);
    }
}
