// W4A4 GEMM for at most 16 rows, as fragments 32 (the decode step): weight streaming, 0.52 bytes per weight.
//
// There are too few outputs to fill the chip with one accumulation chain per wave, and the fp32 chain over
// groups cannot be split.  The exact group sums can: in a round the 8 waves of a workgroup take U groups
// each (group r0 + 8 u + w for wave w: all their loads in flight together), park their 16 x 16 sums in
// LDS, and one thread per output then runs the fp32 chain over those 8 U groups in ascending order -- the
// same bits as the tiled kernel.  Weights and activations are e4m3 numbers, (c + 8) / 512 and a / 512 (rows in the A6 format
// e2m3 ones, as in gemm.hip; the products wait for the weights either way): one
// v_mfma_f32_16x16x128_f8f6f4 per group and 16 columns, one more against the constant -8 per group.  A nibble c + 8 in the low half of
// a byte is the e4m3 number (c + 8) / 512.
// Packed activations carry the same offset, (a + 8)(w + 8) - 8 (a + 8) - 8 (w + 8) + 64 = a w, and need one more
// constant product per group and 16 columns: that costs less than reading them as bytes (every CU reads all
// of them; 16 x 4096 x 11008: 11.0 us with byte activations, 9.7 packed).  Inside a layer the quantizer leaves
// them as the fragments that the lanes want: a KB of 16 different rows takes the CU 27 ns to load, a contiguous
// one 7 (16 x 12288 x 4096: 8.6 -> 7.8 us).
// NB = 16-column blocks per workgroup, RB = 16-row blocks.  With 17 to 32 rows the tiles of gemm.hip start 64 workgroups for
// 4096 columns: 32 x 4096 x 11008 22 us and 13.7 here, 32 x 4096 x 4096 11.0 and 8.5; a 7B decode layer at batch 32 100 -> 71 us
// (a GQA one of 3584 channels 118 -> 79).
//
// Few rows (MODE > FRAG) also bring their own quantizer: every workgroup normalises / quantizes
// the whole rows for itself while its first weights are on their way.  That is a few thousand elements per
// row, read from L2, against a launch and a pass of 16 workgroups that cost 4 to 5 us; from five rows on
// the repeated work costs more than the launch.  SiLU(gate) * up is not among it: 256 workgroups made the same 11008
// products in front of the down projection, 4.7 us of its 11; the gate/up projection makes each once (GLU).
//
// A row's 101 MB of weights of a 7B layer would pass in 18 us: what is left of the 33 that the four launches take is their
// latencies, in this order the rows, their quantizer, the weights, the exchange and the chain.  Rows first
// (weights()), sums and scales of 8 groups in one trip to LDS, and four groups per wave in flight over long rows: down
// 11.2 -> 7.9 us, O 5.4 -> 4.8.  More than 32 KB of weights in flight per workgroup holds the rows up
// instead (QKV 96 KB: 9.6 us, 64 KB 9.4; gate/up 192 KB: 13.5 and 11.4).
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "gemm_common.h"
#include "ldsgrant.h"

namespace {

enum { ROWS_A6 = 0, ROWS_PACKED, ROWS_FRAG, ROWS_QUANT, ROWS_RMSNORM };

struct RowsIn {
    const uint8_t *qa;          // A6 / PACKED / FRAG: activations and token scales
    const float *sa;
    const f16 *x;               // QUANT, RMSNORM: rows [M][K]
    const float *gamma;         // RMSNORM
    float eps;
};

constexpr int RT_THREADS = 512;

// The rows' quantizer: 8 / rows (rounded to a power of two) waves per row, a thread caches its NC chunks of 8
// channels; the same arithmetic as the row kernels in quant.hip.  Leaves e4m3 rows of `stride` bytes and
// the token scales in LDS.  fetch() sets off the first weights, behind the loads that the rows wait for.
// Everything waits for it, so its chain is short: no integer division, a barrier each for the sum and the maximum and one trip to LDS
// of two numbers a lane, what does not depend on the row ahead of it, 1 / sqrt by inv_sqrt, 7 / absmax by sevenths, codes that the
// conversion rounds: a 7B decode step of one row over 32 layers 1247 -> 1150 us, four GQA rows over a long context 67.7 -> 64.4.
template <int MODE, int NC, typename Fetch>
__device__ __forceinline__ void quantize_rows(const RowsIn &in, int M, int K, int G, uint8_t *codes, int stride,
                                              float *scales, double *red, Fetch fetch)
{
    const int shift = M == 1 ? 3 : M == 2 ? 2 : 1, wpr = 1 << shift;     // waves per row
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, row = wave >> shift, part = wave & (wpr - 1);
    const int T = 64 * wpr, idx = part * 64 + lane, nchunk = K >> 3;
    const bool live = row < M;
    const int r = live ? row : M - 1;
    // The weights are asked for behind all waves' loads of the rows, which would else queue behind other waves' weights.
    auto weights = [&] {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        fetch();
    };
    Pack16 v[NC];
    float a = 0.0f;
    double ss = 0.0;
    const uint4 *xr = reinterpret_cast<const uint4 *>(in.x + (size_t)r * K);
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c].u = xr[min(idx + T * c, nchunk - 1)];
    if (MODE != ROWS_RMSNORM) weights();
    // (a clamped chunk repeats one of the row's: harmless for a maximum, left out of the sum)
    if (MODE == ROWS_RMSNORM) {
        constexpr bool EARLY = NC <= 3;                     // the gains of wider shares do not fit beside the rows
        float4 ga[NC][2];
#pragma unroll
        for (int c = 0; EARLY && c < NC; ++c) {
            const float4 *gp = reinterpret_cast<const float4 *>(in.gamma + 8 * min(idx + T * c, nchunk - 1));
            ga[c][0] = gp[0];
            ga[c][1] = gp[1];
        }
        weights();
        double per_channel = 1.0 / (double)K, eps = (double)in.eps;
        asm volatile("" : "+v"(per_channel), "+v"(eps));
        __builtin_amdgcn_sched_barrier(0);                  // (here, while the rows are on their way)
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (idx + T * c < nchunk)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const double f = (double)(float)v[c].h[e];
                    ss = __builtin_fma(f, f, ss);
                }
        waves_max_sum<false, true, true>(a, ss, red, nullptr, wave, row << shift, wpr);
        const float rn = inv_sqrt(ss * per_channel + eps);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (!EARLY) {
                const float4 *gp = reinterpret_cast<const float4 *>(in.gamma + 8 * min(idx + T * c, nchunk - 1));
                ga[c][0] = gp[0];
                ga[c][1] = gp[1];
            }
            const float gm[8] = {ga[c][0].x, ga[c][0].y, ga[c][0].z, ga[c][0].w, ga[c][1].x, ga[c][1].y, ga[c][1].z, ga[c][1].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float hn = (float)v[c].h[e] * rn;
                hn = hn * gm[e];
                v[c].h[e] = to_f16(hn);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf((float)v[c].h[e]));
    waves_max_sum<true, false, true>(a, ss, nullptr, reinterpret_cast<uint32_t *>(red + 32), wave, row << shift, wpr);
    float s, inv;
    sevenths(a, s, inv);
    const float inv_unit = inv * (1.0f / 512.0f);                // (exact)
    if (live) {
        if (idx == 0) scales[row] = s;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int i = idx + T * c;
            if (i < 16 * G) {
                float unit[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) unit[e] = fmaxf((float)v[c].h[e] * inv_unit, -8.0f / 512.0f);      // (as quantize_cached_row)
                const uint2 b = units_to_e4m3(unit);
                *reinterpret_cast<uint2 *>(codes + (size_t)row * stride + 8 * i) = i < nchunk ? b : make_uint2(0, 0);
            }
        }
    }
    __syncthreads();
}

// 32 packed codes c as the e4m3 bytes (c + 8) / 512, evens and odds of each dword apart
__device__ __forceinline__ void unsigned_e4m3(const uint4 &p, uint4 &lo, uint4 &hi)
{
    const uint32_t w[4] = {p.x, p.y, p.z, p.w};
    uint32_t o[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[2 * i] = (w[i] & 0x0F0F0F0Fu) ^ 0x08080808u;
        o[2 * i + 1] = ((w[i] >> 4) & 0x0F0F0F0Fu) ^ 0x08080808u;
    }
    lo = make_uint4(o[0], o[1], o[2], o[3]);
    hi = make_uint4(o[4], o[5], o[6], o[7]);
}

// GLU: the columns are gate | up, NB = 2 and a workgroup has 16 of each, of the same channels: it stores SiLU(gate) * up of
// their fp16 roundings, y is [M][N / 2].
// RB: 16-row blocks, 2 for fragments of 17 to 32 rows: a weight read serves both.
// RES: residuals are added.
template <int NB, int U, int MODE, int NC, bool GLU, int RB, bool RES>
__global__ __launch_bounds__(RT_THREADS, 4) void w4a4_rows16_kernel(
    const uint4 *__restrict__ wp, const f16 *__restrict__ sw, const void *rows, const float *beside, int M, int N, int K, int G,
    f16 *__restrict__ y, int ldy, const f16 *__restrict__ res, int ldr, float eps, int code_stride)
{
    // (plain arguments, those of the first loads in front: they are in registers when a wave starts)
    const RowsIn in = {(const uint8_t *)rows, beside, (const f16 *)rows, beside, eps};
    constexpr int R = 8 * U;                        // groups per round
    constexpr int SD = 8 * NB * R;                  // scale dwords (two columns of a group) per round
    constexpr int SPT = (SD + RT_THREADS - 1) / RT_THREADS;
    constexpr int SROW = R + 8;                     // halves per column of staged scales (16-byte pieces, padded)
    constexpr bool FEW = MODE > ROWS_FRAG;          // at most 4 rows: lanes 0 to 15 hold the sums that count
    constexpr int XS = FEW ? 64 : 256;              // sums of a group and block
    constexpr int OPT = GLU || RB == 2 ? NB : 1;    // outputs per owner thread
    constexpr int BUF = R * NB * RB * XS + 8 * NB * SROW;   // floats of one exchange buffer
    static_assert(!(RES && (GLU || MODE == ROWS_RMSNORM)), "(never together)");
    static_assert((NB <= 2 || (FEW && !GLU)) && (!GLU || NB == 2) && (RB == 1 || (RB == 2 && MODE == ROWS_FRAG)), "an owner per output");
    extern __shared__ __align__(16) uint4 lds_rows[];
    float *xbuf = reinterpret_cast<float *>(lds_rows);      // 2 x { sums [R][NB][4][64]; scales f16 [16 NB][SROW] }
    float *row_scale = xbuf + 2 * BUF;                                            // [16]
    double *red = reinterpret_cast<double *>(row_scale + 16);                     // [48]: sums, maxima
    uint8_t *codes = reinterpret_cast<uint8_t *>(red + 48);                       // [M][code_stride], MODE > FRAG
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // chain ownership: thread t owns the output(s) held by (block t / XS, or both for GLU and of row block t / XS for RB = 2;
    // register oreg, lane ol)
    const int oi = RB == 2 ? tid / XS : 0, oj = GLU || RB == 2 ? 0 : tid / XS, oreg = tid / (XS / 4) & 3, ol = tid % (XS / 4);
    const bool owner = XS * NB * RB / OPT >= RT_THREADS || tid < XS * NB * RB / OPT;
    const int om = 16 * oi + 4 * (ol >> 4) + oreg;
    const int C = GLU ? N >> 1 : N;                 // output columns
    const int up = GLU ? C : 16;                    // from a column of the first block to the second's
    float y32[OPT];
#pragma unroll
    for (int o = 0; o < OPT; ++o) y32[o] = 0.0f;

    constexpr bool E2M3 = MODE == ROWS_A6;
    constexpr float UNIT = E2M3 ? F6_UNIT : F8_UNIT;
    constexpr int FMT = E2M3 ? 2 : 0;               // of the matrix instruction's operands
    const int arow_at = min(c16, M - 1);
    const uint8_t *arow = MODE == ROWS_PACKED ? in.qa + (size_t)arow_at * (K >> 1)
                          : E2M3 ? in.qa + (size_t)(arow_at >> 2) * quota_a6_groups(G) * 384 + (arow_at & 3) * 64 : nullptr;
    uint32_t flip[3];
    if (E2M3) e2m3_flips(flip);
    uint4 ra[U][MODE == ROWS_A6 ? 2 : RB], rb[U][NB];
    uint32_t rsv[SPT];
    auto fetch = [&](int n0, int r0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = min(r0 + 8 * u + wave, G - 1);
            const uint4 *wg = wp + ((size_t)g * N + n0) * 4;
#pragma unroll
            for (int j = 0; j < NB; ++j) rb[u][j] = wg[4 * j * up + 4 * c16 + q];
            if (MODE == ROWS_FRAG) {
#pragma unroll
                for (int i = 0; i < RB; ++i) ra[u][i] = *reinterpret_cast<const uint4 *>(in.qa + (size_t)(i * G + g) * 1024 + 16 * lane);
            } else if (MODE == ROWS_A6) {
                ra[u][0] = *reinterpret_cast<const uint4 *>(arow + g * 384 + 16 * q);
                const uint2 t = *reinterpret_cast<const uint2 *>(arow + g * 384 + 256 - 32 * (arow_at & 3) + 8 * q);
                ra[u][MODE == ROWS_A6 ? 1 : 0] = make_uint4(t.x, t.y, 0, 0);
            } else if (MODE == ROWS_PACKED) {
                ra[u][0] = *reinterpret_cast<const uint4 *>(arow + min(g * 64 + q * 16, (K >> 1) - 16));
            }
        }
#pragma unroll
        for (int k = 0; k < SPT; ++k) {
            const int d = min(tid + RT_THREADS * k, SD - 1), g = min(r0 + d / (8 * NB), G - 1);
            rsv[k] = *reinterpret_cast<const u32_at2 *>(sw + (size_t)g * N + n0 + (GLU ? d / 8 % NB * up + 2 * (d % 8) : 2 * (d % (8 * NB))));
        }
    };
    constexpr int BC = GLU ? 16 : 16 * NB;          // output columns per workgroup
    const int nblk = C / BC;
    int blk = blockIdx.x, r0 = 0, par = 0, grid = gridDim.x;
    // What the outputs take besides the sums is asked for with their first weights, not at the end of their chain.  Every thread
    // asks for the same, so that the loads in flight can be counted; a launch without residuals is an instantiation without these
    // loads (weight scales in their place, for the count: fragments 16 x 12288 x 4096 7.0 us, 7.6 so, four rows with their RMSNorm 10.7, 11.0).
    f16 rsd[RES ? OPT : 1];
    float sa_out = 0.0f;
    const int om_in = min(om, M - 1);
    auto residuals = [&](int b) {
        if constexpr (RES) {
            const f16 *rp = res + (size_t)om_in * ldr;
#pragma unroll
            for (int o = 0; o < OPT; ++o) rsd[o] = rp[b * BC + 16 * min(o + oj, NB - 1) + (ol & 15)];
        }
    };
    // where this thread leaves a round's scales and finds those and the sums of its outputs
    int scale_at[SPT], codes_at, chain_scales, chain_sums;
    auto places = [&] {
        codes_at = arow_at * code_stride + 32 * q;
        chain_scales = (16 * oj + (ol & 15)) * SROW;
        chain_sums = (oj * RB + oi) * XS + oreg * (XS / 4) + ol;
#pragma unroll
        for (int k = 0; k < SPT; ++k) {
            const int d = tid + RT_THREADS * k;
            scale_at[k] = 2 * (d % (8 * NB)) * SROW + d / (8 * NB);
        }
    };
    if constexpr (GLU) places();
    if constexpr (MODE > ROWS_FRAG)
        quantize_rows<MODE, NC>(in, M, K, G, codes, code_stride, row_scale, red, [&] {
            fetch(blk * BC, 0);
            residuals(blk);
            // (these come here, behind the loads, not in front of the weights or between the quantizer and the first product: a 7B decode
            // step of one row over 32 layers 1153 -> 1136 us; gate/up, whose share is longer, takes 1 % less with its own in front)
            if constexpr (!GLU) {
                __builtin_amdgcn_sched_barrier(0);
                places();
            }
            asm volatile("" : "+s"(ldy), "+s"(grid), "+v"(codes_at), "+v"(chain_scales), "+v"(chain_sums));
#pragma unroll
            for (int k = 0; k < SPT; ++k) asm volatile("" : "+v"(scale_at[k]));
        });
    else {
        fetch(blk * BC, 0);
        residuals(blk);
        sa_out = in.sa[om_in];
        if constexpr (!GLU) places();
    }
    const i32x8 minus8 = E2M3 ? i32x8{(int)0x28A28A28, (int)0x8A28A28A, (int)0xA28A28A2, (int)0x28A28A28, (int)0x8A28A28A, (int)0xA28A28A2, 0, 0} : i32x8{(int)0x88888888, (int)0x88888888, (int)0x88888888, (int)0x88888888,
                               (int)0x88888888, (int)0x88888888, (int)0x88888888, (int)0x88888888};
    while (true) {                                  // rounds of this workgroup's column blocks
        float *accs = xbuf + par * BUF;
        f16 *scs = reinterpret_cast<f16 *>(accs + R * NB * RB * XS);
        f32x4 acc[U][NB][RB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            constexpr bool OFFSET_A = MODE == ROWS_PACKED || MODE == ROWS_FRAG;
            const float c0 = OFFSET_A ? 64.0f * 128.0f / F8_UNIT : 0.0f;
            i32x8 fa[RB];
            f32x4 k4[RB];
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                uint4 a0, a1;
                if constexpr (MODE == ROWS_A6) {
                    a0 = ra[u][0];
                    a1 = ra[u][1];
                } else if constexpr (OFFSET_A) {
                    unsigned_e4m3(ra[u][i], a0, a1);
                } else {
                    const int g = min(r0 + 8 * u + wave, G - 1);
                    const uint4 *ag = reinterpret_cast<const uint4 *>(codes + codes_at + g * 128);
                    a0 = ag[0];
                    a1 = ag[1];
                }
                fa[i] = i32x8{(int)a0.x, (int)a0.y, (int)a0.z, (int)a0.w, (int)a1.x, (int)a1.y, (int)a1.z, (int)a1.w};
                k4[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[i], minus8, f32x4{c0, c0, c0, c0}, FMT, FMT, 0, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                i32x8 fb;
                if constexpr (E2M3) {
                    weights_e2m3(rb[u][j], flip, fb);
                } else {
                    uint4 b0, b1;
                    unsigned_e4m3(rb[u][j], b0, b1);
                    fb = i32x8{(int)b0.x, (int)b0.y, (int)b0.z, (int)b0.w, (int)b1.x, (int)b1.y, (int)b1.z, (int)b1.w};
                }
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    f32x4 k = k4[i];
                    if (OFFSET_A) k = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(minus8, fb, k, 0, 0, 0, 0, 0, 0);
                    acc[u][j][i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[i], fb, k, FMT, FMT, 0, 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < SPT; ++k) {             // this round's scales -> LDS, [column][group]
            const int d = tid + RT_THREADS * k;
            if (SD % RT_THREADS == 0 || d < SD) {
                union { uint32_t w; f16 h[2]; } t;
                t.w = rsv[k];
                scs[scale_at[k]] = t.h[0];
                scs[scale_at[k] + SROW] = t.h[1];
            }
        }
        const bool last = r0 + R >= G;
        const int nblk_next = last ? blk + grid : blk, r_next = last ? 0 : r0 + R;
        if (nblk_next < nblk) fetch(nblk_next * BC, r_next);       // the next loads fly during the exchange
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int b = 0; b < RB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (!FEW || lane < 16) accs[(((8 * u + wave) * NB + j) * RB + b) * XS + i * (XS / 4) + lane] = acc[u][j][b][i];
        __syncthreads();        // (the other buffer's readers passed the one before)
        if (owner) {
#pragma unroll
            for (int o = 0; o < OPT; ++o) {
                const Pack16 *sp = reinterpret_cast<const Pack16 *>(scs + chain_scales + 16 * o * SROW);
                const float *ap = accs + chain_sums + o * RB * XS;
#pragma unroll
                for (int i8 = 0; i8 < U; ++i8) {
                    if (!FEW && r0 + 8 * i8 >= G) break;
                    const Pack16 s8 = sp[i8];
                    float sum[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) sum[i] = ap[(8 * i8 + i) * NB * RB * XS];
                    __builtin_amdgcn_sched_barrier(0);          // one trip to LDS, not one per pair
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        y32[o] = __builtin_fmaf(sum[i], r0 + 8 * i8 + i < G ? (float)s8.h[i] : 0.0f, y32[o]);
                }
            }
            if (last) {
                if (om < M) {
                    const float sa = MODE <= ROWS_FRAG ? sa_out : row_scale[om];
#pragma unroll
                    for (int o = 0; o < (GLU ? 1 : OPT); ++o) {
                        const int on = blk * BC + 16 * (o + oj) + (ol & 15);
                        float v = y32[o] * (sa * UNIT);
                        if constexpr (RES) v = v + (float)rsd[o];
                        f16 out = to_f16(v);
                        if (GLU) out = silu_mul((float)out, (float)to_f16(y32[OPT - 1] * (sa * UNIT)));
                        y[(size_t)om * ldy + on] = out;
                    }
                }
#pragma unroll
                for (int o = 0; o < OPT; ++o) y32[o] = 0.0f;
            }
        }
        if (nblk_next >= nblk) break;
        if (last) residuals(nblk_next);
        blk = nblk_next;
        r0 = r_next;
        par ^= 1;
    }
}

// PER_CU: workgroups wanted per CU.  A launch asks for no more than the LDS has room for: what is left over would run in a
// second round and quantize the rows once more.  <2, 2> takes 19.6 KB, 68.8 without a quantizer, and 128 G + 16
// bytes a row.
template <int NB, int U, int PER_CU, int MODE, int NC, bool GLU = false, int RB = 1>
int launch_rows16(const RowsIn &in, int M, const quota_weights *W, f16 *y, int ldy, const f16 *res, int ldr,
                  int code_stride, hipStream_t st)
{
    constexpr int R = 8 * U;
    const int G = (W->K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    const size_t lds = 2 * (R * NB * RB * (MODE > ROWS_FRAG ? 256 : 1024) + 16 * NB * (R + 8) * 2) + 64 + 384 + (MODE > ROWS_FRAG ? (size_t)M * code_stride : 0);
    const double Md = M, Nd = W->N, Kd = W->K;
    ProfScope prof(QUOTA_K_GEMM_ROWS16, 2.0 * Md * Nd * Kd,
                   Nd * Kd / 2 + 2.0 * Nd * G + Md * Kd / 2 + 4 * Md + (GLU ? 1.0 : 2.0) * Md * Nd * (res ? 2 : 1), st);
    const int per_cu = min(PER_CU, (int)(160 * 1024 / lds));
    auto run = [&](auto with_res) {
        constexpr auto kernel = w4a4_rows16_kernel<NB, U, MODE, NC, GLU, RB, decltype(with_res)::value>;
        if (!grant_lds<kernel>()) return false;
        kernel<<<dim3(min(W->N / (16 * NB), 256 * per_cu)), dim3(RT_THREADS), lds, st>>>(
            (const uint4 *)W->packed, (const f16 *)W->scales, MODE > ROWS_FRAG ? (const void *)in.x : in.qa, MODE > ROWS_FRAG ? in.gamma : in.sa, M, W->N, W->K, G, y,
            ldy, res, ldr, in.eps, code_stride);
        return true;
    };
    bool granted;
    if constexpr (GLU || MODE == ROWS_RMSNORM) granted = run(std::false_type());
    else if constexpr (MODE == ROWS_QUANT) granted = run(std::true_type());
    else granted = res ? run(std::true_type()) : run(std::false_type());
    if (!granted) return QUOTA_ERR_HIP;
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

// 16 columns per workgroup up to 4096 columns (256 workgroups: one per CU), with two groups per wave in flight, four
// over long rows, which stream longer than they start up; 32 beyond, two groups up to 8192 columns (at
// most one workgroup per CU again), else three workgroups per CU with one group per wave, or, with a quantizer in
// front, two per CU (one, where the rows leave no room for two) with two, so that fewer repeat its work (one row, gate/up
// of 22016 columns: 10.8 us inside with two per CU, 12.8 with one, 13.8 with three).  One or two rows take 48 columns where
// that is one share for every CU and 32 are more, so that no CU has two (1 x 12288 x 4096 9.6 -> 8.4 us, 2 x 9216 x 6144
// 12.4 -> 10.9, 1 x 8448 x 8192 13.2 -> 11.6; with three rows whose quantizer one workgroup per CU does alone a layer takes 1 %
// longer; six chunks of a row per thread leave no registers for it: 2 x 12288 x 8192 18.0 us, 17.0 to 17.7 with 32 columns).
// Workgroups walk over the columns.
// Short rows end in their first round, half of which is empty with two groups per wave: one per wave for up to 8 groups, us: 1 x 1536 x 512
// 3.10 -> 2.96, 1 x 6144 x 768 3.63 -> 3.19, 4 x 1024 x 1024 2.79 -> 2.59, fragments 16 x 1536 x 512 2.44 -> 2.24 (1 x 12288 x 1024,
// more columns than the chip takes at once, 4.00 and 4.08).  Gate/up up to 16 groups and a column block for each of 512 workgroups: 1 x 2752 x 512
// 3.47 -> 3.08, 1 x 11008 x 2048 5.54 -> 4.96, 16 x 8192 x 2048 4.20 -> 3.82 (4 x 22016 x 2048 8.93 and 10.11).
// Packed, 16 rows, us at 4096 x 11008 / 5120 x 13824 / 22016 x 4096: <1, 2> 9.6 / 16.0 / 16.5, <1, 4> 9.3 / 17.5 / 17.3,
// <2, 2> 11.6 / 13.7 / 13.2, <2, 1> 12.4 / 15.4 / 12.9.
template <int MODE, int NC, int RB = 1>
int rows16(const RowsIn &in, int M, const quota_weights *W, f16 *y, int ldy, const f16 *res, int ldr, int code_stride,
           hipStream_t st)
{
    if constexpr (NC == 1)
        if (W->K <= 1024 && W->N <= 8192) {
            if (W->N <= 4096) return launch_rows16<1, 1, 1, MODE, NC, false, RB>(in, M, W, y, ldy, res, ldr, code_stride, st);
            return launch_rows16<2, 1, 2, MODE, NC, false, RB>(in, M, W, y, ldy, res, ldr, code_stride, st);
        }
    if (W->N <= 4096) {
        if constexpr (MODE != ROWS_RMSNORM && !(MODE == ROWS_QUANT && NC == 1))      // (one chunk: 4096 channels at most)
            if (W->K > 8192) return launch_rows16<1, 4, 1, MODE, NC, false, RB>(in, M, W, y, ldy, res, ldr, code_stride, st);
        return launch_rows16<1, 2, 1, MODE, NC, false, RB>(in, M, W, y, ldy, res, ldr, code_stride, st);
    }
    if constexpr (MODE == ROWS_RMSNORM && NC <= 3)
        if (M <= 2 && W->N > 8192 && W->N <= 48 * 256 && W->N % 48 == 0)
            return launch_rows16<3, 2, 1, MODE, NC>(in, M, W, y, ldy, res, ldr, code_stride, st);
    if constexpr (MODE <= ROWS_FRAG)
        if (W->N > 8192) return launch_rows16<2, 1, 3, MODE, NC, false, RB>(in, M, W, y, ldy, res, ldr, code_stride, st);
    return launch_rows16<2, 2, 2, MODE, NC, false, RB>(in, M, W, y, ldy, res, ldr, code_stride, st);
}

template <int MODE, int NC, int RB = 1>
int rows16_glu(const RowsIn &in, int M, const quota_weights *W, f16 *z, int code_stride, hipStream_t st)
{
    const int F = W->N / 2;
    if constexpr (MODE <= ROWS_FRAG)
        if (W->N > 8192) return launch_rows16<2, 1, 3, MODE, NC, true, RB>(in, M, W, z, F, nullptr, 0, code_stride, st);
    if constexpr (NC <= 3)
        if (W->K <= 2048 && W->N <= 16384) return launch_rows16<2, 1, 2, MODE, NC, true, RB>(in, M, W, z, F, nullptr, 0, code_stride, st);
    return launch_rows16<2, 2, 2, MODE, NC, true, RB>(in, M, W, z, F, nullptr, 0, code_stride, st);
}

// run(chunks per thread, bytes of a row of codes in LDS)
template <typename RUN>
int rows16_quantizing(int M, int K, RUN run)
{
    const int G = (K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W, T = M == 1 ? 512 : M == 2 ? 256 : 128;
    const int nc = (16 * G + T - 1) / T;                  // 8-channel chunks per thread
    const int stride = G * 128 + 16;                      // 16 more: rows start on different LDS banks
    if (nc <= 1) return run(std::integral_constant<int, 1>(), stride);
    if (nc <= 3) return run(std::integral_constant<int, 3>(), stride);
    return run(std::integral_constant<int, 6>(), stride);
}

}  // namespace

bool quota_internal_rows16_quantizes(int M, int K)
{
    const int G = (K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W, T = M == 1 ? 512 : M == 2 ? 256 : 128;
    return M <= 4 && (16 * G + T - 1) / T <= 6;            // six chunks of a row per thread fit in registers
}

int quota_internal_rows16(const uint8_t *qa, quota_rows16_format format, const float *sa, int M, const quota_weights *W, void *y, int ldy,
                          const void *res, int ldr, hipStream_t st)
{
    RowsIn in = {};
    in.qa = qa;
    in.sa = sa;
    switch (format) {
    case QUOTA_ROWS16_A6: return rows16<ROWS_A6, 1>(in, M, W, (f16 *)y, ldy, (const f16 *)res, ldr, 0, st);
    case QUOTA_ROWS16_FRAG:
        if (M > 16) return rows16<ROWS_FRAG, 1, 2>(in, M, W, (f16 *)y, ldy, (const f16 *)res, ldr, 0, st);
        return rows16<ROWS_FRAG, 1>(in, M, W, (f16 *)y, ldy, (const f16 *)res, ldr, 0, st);
    default: return rows16<ROWS_PACKED, 1>(in, M, W, (f16 *)y, ldy, (const f16 *)res, ldr, 0, st);
    }
}

int quota_internal_rows16_frag_silu(const uint8_t *qf, const float *sa, int M, const quota_weights *W, void *z, hipStream_t st)
{
    RowsIn in = {};
    in.qa = qf;
    in.sa = sa;
    return M > 16 ? rows16_glu<ROWS_FRAG, 1, 2>(in, M, W, (f16 *)z, 0, st) : rows16_glu<ROWS_FRAG, 1>(in, M, W, (f16 *)z, 0, st);
}

int quota_internal_rows16_quantize(const void *x, int M, const quota_weights *W, void *y, int ldy, const void *res,
                                   int ldr, hipStream_t st)
{
    if (!res) return QUOTA_ERR_NULL;                      // (the projections that add one)
    RowsIn in = {};
    in.x = (const f16 *)x;
    return rows16_quantizing(M, W->K, [&](auto nc, int stride) {
        return rows16<ROWS_QUANT, nc()>(in, M, W, (f16 *)y, ldy, (const f16 *)res, ldr, stride, st);
    });
}

int quota_internal_rows16_rmsnorm(const void *x, const float *gamma, float eps, int M, const quota_weights *W, void *y,
                                  int ldy, bool glu, hipStream_t st)
{
    RowsIn in = {};
    in.x = (const f16 *)x;
    in.gamma = gamma;
    in.eps = eps;
    return rows16_quantizing(M, W->K, [&](auto nc, int stride) {
        if (glu) return rows16_glu<ROWS_RMSNORM, nc()>(in, M, W, (f16 *)y, stride, st);
        return rows16<ROWS_RMSNORM, nc()>(in, M, W, (f16 *)y, ldy, nullptr, 0, stride, st);
    });
}
