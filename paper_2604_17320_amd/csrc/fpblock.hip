// Sensitivity profiling for the offline allocator (Eq. 1): the full-precision counterpart of a
// decoder block -- fp16 storage, fp32 accumulation, no quantizer anywhere -- the per-sample
// deviation norms ||x^q - x||_2 and ||x||_2, and the call that runs a block both ways on one
// input.  Calibration-time code, outside the deployed forward pass, but a calibration runs it for
// every layer and sample: its time is the fp16 GEMMs'.
#include <type_traits>
#include "common.h"
#include "internal.h"
#include "gemm_common.h"
#include "ldscopy.h"

namespace {

// silu(gate) * up of eight channels, the product rounded to fp32 and that to fp16
__device__ __forceinline__ Pack16 silu_mul_fp(Pack16 g, const Pack16 &u)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float gv = (float)g.h[e];
        g.h[e] = to_f16(gv / (1.0f + expf(-gv)) * (float)u.h[e]);
    }
    return g;
}
// Rotate-half RoPE of eight channels x of a head, whose partners half a head away are xp; cp, sp: the angles of their pairs
__device__ __forceinline__ Pack16 rope_fp(Pack16 x, const Pack16 &xp, const float *cp, const float *sp, bool second)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const f32x4 cs = *reinterpret_cast<const f32x4_at4 *>(cp + 4 * i), sn = *reinterpret_cast<const f32x4_at4 *>(sp + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float a = (float)x.h[4 * i + e] * cs[e], b = (float)xp.h[4 * i + e] * sn[e];
            x.h[4 * i + e] = (f16)(second ? a + b : a - b);
        }
    }
    return x;
}

// ---- y = x W^T (+ residual): fp16 operands, fp32 accumulation, fp16 result ------------------
// WM x WN waves cover a tile, each 32 RT x 32 CT of it by v_mfma_f32_32x32x16_f16.  Both operands come to LDS 64
// channels at a time by asynchronous copies into a ring of RING stages, all but the current one on their way while it
// is multiplied; a stage costs one counted wait and one barrier.  What binds it is the round trip of a stage:
// two workgroups of 128 x 128 on a CU with one stage on its way each left the waves waiting for 44 % of their
// lives, and a launch that gives a CU one took as long as two (640 x 4096 x 4096 65 us).  A workgroup that has the
// CU to itself, 8 waves and two to five stages on their way (one for 256 and 320 x 256) does it in 39, and leaves the choice of the tile to the
// number of workgroups.  The next step's fragments are read, and a stage's copies started, between the products of
// the current one (SPREAD: over how many of the stage's 4 steps; all at once they hold the address unit up: 1280 x 4096 x
// 11008 178 us with one stage on its way, 160 spread over three steps and two on their way).  1280 rows: 1.06 PFLOP/s at 12288 x 4096,
// 0.99 at 22016 x 4096 (0.99 and 0.97 with RoPE and the SiLU product), 0.70 and 0.73 at 4096 x 4096 and 4096 x 11008 (0.91, 0.86, 0.62 and 0.67 before).
// LDS rows are 128 bytes, 16-byte piece p of row r at p ^ (r % 8).
// Lane l supplies 8 consecutive k of row (l % 32) to both operands (k slots 8 (l / 32) .. +7 of the
// step), and receives column l % 32 of the tile, rows 8 (r / 4) + 4 (l / 32) + r % 4 for r = 0..15.
// Rows beyond M and N repeat the last one and are not stored.  Needs N % 64 == 0, K % 16 == 0, x and W at
// multiples of 16 bytes; residual and y may lie anywhere.
// What is made of the result in front of the store, of its fp16 roundings (as launches of their own RoPE and the SiLU product took 17 us each for 1280
// rows of the 7B shape and a second trip of q | k | v and gate | up through memory; the block and its low-bit one 1012 -> 994 us):
struct FpPlain {};                       // nothing
struct FpSilu {};                        // W's rows are gate | up: y [M][N / 2] = silu(gate) * up, a tile has as many columns of both
struct FpRope {                          // N is q | k | v: q and k rotated by halves of a head at the tokens' position ids
    const int32_t *pos;
    const float *cosT, *sinT;
    int n_pos, d, dkv, dh;
    f16 *q, *k, *v;
};
template <int WM, int WN, int RT, int CT, int RING, int SPREAD, typename EPI>
__global__ __launch_bounds__(64 * WM * WN, 2) void fp_gemm_kernel(const f16 *__restrict__ x, int M, int K,
                                                                    const f16 *__restrict__ W, int N,
                                                                    const f16 *__restrict__ residual,
                                                                    f16 *__restrict__ y, int tiles_m, int tiles_n, EPI epi)
{
    constexpr bool SILU = std::is_same_v<EPI, FpSilu>, ROPE = std::is_same_v<EPI, FpRope>;
    constexpr int NW = WM * WN, NT = 64 * NW, BM = 32 * RT * WM, BN = 32 * CT * WN;
    constexpr int KS = 64, PR = KS / 8, STG = (BM + BN) * PR, COPIES = STG / NT;       // a stage in 16-byte pieces, pieces per thread
    constexpr int FROW = BN + 4;                                // floats per staged output row
    static_assert(STG % NT == 0 && RING >= 2 && 32 * WM * (BN / 8) % NT == 0, "whole pieces per thread, copies in flight");
    constexpr int STRIP = 32 * WM * FROW / 4;
    __shared__ uint4 lds[RING * STG > STRIP ? RING * STG : STRIP];      // [stage][x rows, W rows][8]
    const unsigned lds0 = lds_address(lds);
    int tm, tn;
    tile_of(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
    // this thread's pieces of a stage: rows (tid + NT j) / 8 of x, then W
    unsigned row_at[COPIES], piece[COPIES];
#pragma unroll
    for (int j = 0; j < COPIES; ++j) {
        const int r = (tid + NT * j) / PR;
        int w = min(n0 + r - BM, N - 1) - n0;
        if (SILU) w = min(n0 / 2 + (r - BM) % (BN / 2), N / 2 - 1) - n0 / 2;       // gate rows, then up rows of the same channels
        row_at[j] = 2u * (unsigned)(r < BM ? min(m0 + r, M - 1) - m0 : w) * (unsigned)K;
        piece[j] = 16 * ((tid & 7) ^ (r & 7));
    }
    const f16 *xb = x + (size_t)m0 * K, *wb = W + (size_t)(SILU ? n0 / 2 : n0) * K;
    const size_t up = SILU ? (size_t)(N / 2) * K : 0;            // from a gate row to its up row
    const int stages = (K + KS - 1) / KS;
    auto load = [&](int stage, int slot, int from, int to) {
        const int k0 = KS * min(stage, stages - 1);                     // (stages past the end keep the count of copies)
        const unsigned left = 2u * (unsigned)(K - k0) - 16;             // last whole piece of a row (a ragged end repeats it)
#pragma unroll
        for (int j = from; j < to; ++j) {
            const int first = 64 / PR * (wave + NW * j);                // row of the copy
            copy16_to_lds((first < BM ? xb : wb) + (k0 + (SILU && first >= BM + BN / 2 ? up : 0)), row_at[j] + min(piece[j], left),
                          lds0 + (unsigned)(slot * STG * 16 + (wave + NW * j) * 1024));
        }
    };
    f32x16 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
#pragma unroll
    for (int st = 0; st < RING - 1; ++st) load(st, st, 0, COPIES);
    int slot = 0;
#pragma unroll 1
    for (int st = 0; st < stages; ++st) {
        // this wave's copies of the stage have arrived, RING - 2 later stages may be on their way; behind the barrier so have
        // all waves', and the slot read before it is free
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 2) * COPIES) : "memory");
        __syncthreads();
        const int free = slot ? slot - 1 : RING - 1;
        const uint4 *ax = lds + slot * STG + (32 * RT * wm + l32) * PR, *bx = lds + slot * STG + (BM + 32 * CT * wn + l32) * PR;
        f16x8 a[2][RT], b[2][CT];
        auto fragments = [&](int s) {
            const int p = (2 * s + half) ^ (l32 & 7);
#pragma unroll
            for (int j = 0; j < CT; ++j) b[s & 1][j] = *reinterpret_cast<const f16x8 *>(bx + 32 * PR * j + p);
#pragma unroll
            for (int i = 0; i < RT; ++i) a[s & 1][i] = *reinterpret_cast<const f16x8 *>(ax + 32 * PR * i + p);
        };
        fragments(0);
#pragma unroll
        for (int s = 0; s < KS / 16; ++s) {
            if (s && KS * st + 16 * s >= K) break;
            if (s + 1 < KS / 16) fragments(s + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
#pragma unroll
                for (int j = 0; j < CT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[s & 1][i], b[s & 1][j], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int AT = RT * SPREAD;
                const int t = s * RT + i;
                if (t < AT) load(st + RING - 1, free, COPIES * t / AT, COPIES * (t + 1) / AT);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = slot + 1 < RING ? slot + 1 : 0;
    }
    drain();                                          // (the copies past the end)
    __syncthreads();
    // WM x 32 rows at a time through LDS, so that a thread finishes 8 neighbouring columns of a row
    float *stage = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        if (i) __syncthreads();
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                stage[(32 * wm + 8 * (r >> 2) + 4 * half + (r & 3)) * FROW + 32 * CT * wn + 32 * j + l32] = acc[i][j][r];
        __syncthreads();
        constexpr int WIDTH = SILU ? BN / 2 : BN;               // columns of a row that are stored
        const int n_at = SILU ? n0 / 2 : n0, n_end = SILU ? N / 2 : N;
        // eight staged results, and their fp16 roundings
        auto take = [&](int row, int c, float (&v)[8]) {
            *reinterpret_cast<float4 *>(v) = *reinterpret_cast<const float4 *>(stage + row * FROW + c);
            *reinterpret_cast<float4 *>(v + 4) = *reinterpret_cast<const float4 *>(stage + row * FROW + c + 4);
        };
        auto rounded = [](const float (&v)[8]) {
            Pack16 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o.h[e] = (f16)v[e];
            return o;
        };
#pragma unroll
        for (int k = 0; k < 32 * WM * (WIDTH / 8) / NT; ++k) {
            const int idx = k * NT + tid, row = idx / (WIDTH / 8), c = 8 * (idx % (WIDTH / 8));
            const int m = m0 + 32 * RT * (row >> 5) + 32 * i + (row & 31), n = n_at + c;
            if (m >= M || n >= n_end) continue;
            float v[8];
            take(row, c, v);
            if constexpr (SILU) {
                float up[8];
                take(row, c + BN / 2, up);
                store16_at2(y + (size_t)m * n_end + n, silu_mul_fp(rounded(v), rounded(up)).u);
            } else if constexpr (ROPE) {
                Pack16 o = rounded(v);
                const int hd = epi.dh / 2, in = n & (epi.dh - 1);       // (64 or 128: tiles begin with a head)
                if (n < epi.d + epi.dkv) {
                    float w[8];
                    take(row, in >= hd ? c - hd : c + hd, w);
                    const int p = min(max(epi.pos[m], 0), epi.n_pos - 1);
                    o = rope_fp(o, rounded(w), epi.cosT + (size_t)p * hd + in % hd, epi.sinT + (size_t)p * hd + in % hd, in >= hd);
                }
                f16 *to = n < epi.d ? epi.q + (size_t)m * epi.d + n
                                    : (n < epi.d + epi.dkv ? epi.k + (size_t)m * epi.dkv + n - epi.d
                                                           : epi.v + (size_t)m * epi.dkv + n - epi.d - epi.dkv);
                *reinterpret_cast<uint4 *>(to) = o.u;
            } else {
                if (residual) {
                    Pack16 rv;
                    rv.u = load16_at2(residual + (size_t)m * N + n);
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] += (float)rv.h[e];
                }
                store16_at2(y + (size_t)m * N + n, rounded(v).u);
            }
        }
    }
}

// ---- h = x / sqrt(mean(x^2) + eps) * gamma, one workgroup per row; x and gamma may lie anywhere ----
__global__ __launch_bounds__(256) void fp_rmsnorm_kernel(const f16 *__restrict__ x, int d,
                                                          const float *__restrict__ gamma, float eps,
                                                          f16 *__restrict__ h)
{
    __shared__ float part[4];
    const f16 *row = x + (size_t)blockIdx.x * d;
    uint4 *out = reinterpret_cast<uint4 *>(h + (size_t)blockIdx.x * d);
    float s = 0.0f;
    for (int c = threadIdx.x; c < d >> 3; c += 256) {
        Pack16 v;
        v.u = load16_at2(row + 8 * c);
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (float)v.h[e] * (float)v.h[e];
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    const float inv = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)d + eps);
    for (int c = threadIdx.x; c < d >> 3; c += 256) {
        Pack16 v;
        v.u = load16_at2(row + 8 * c);
        const f32x4_at4 *gm = reinterpret_cast<const f32x4_at4 *>(gamma + 8 * c);
        const f32x4 g[2] = {gm[0], gm[1]};
#pragma unroll
        for (int e = 0; e < 8; ++e) v.h[e] = (f16)((float)v.h[e] * inv * g[e >> 2][e & 3]);
        out[c] = v.u;
    }
}

// ---- Eq. 1 per sample: ||x^q - x||_2 and ||x||_2 over the n values of sample blockIdx.x --------
// gridDim.y workgroups share a sample: with `part` they leave their sums in part[sample][workgroup]
// for deviation_finish_kernel; without it one workgroup does the sample alone (one workgroup pulls
// some 20 GB/s out of memory with 2-byte loads: 1.2 ms for two 640 x 4096 samples, 0.01 ms shared).
constexpr int DEV_PARTS = 64;
__global__ __launch_bounds__(1024) void deviation_kernel(const f16 *__restrict__ xq,
                                                          const f16 *__restrict__ x, long n, int vec,
                                                          double *__restrict__ part_out,
                                                          double *__restrict__ diff_norm,
                                                          double *__restrict__ ref_norm)
{
    __shared__ double part[2][16];
    const f16 *a = xq + (size_t)blockIdx.x * n, *b = x + (size_t)blockIdx.x * n;
    double sd = 0.0, sr = 0.0;
    auto add = [&](f16 av, f16 bv) {
        const double r = (double)(float)bv, e = (double)(float)av - r;
        sd += e * e;
        sr += r * r;
    };
    const long first = (long)blockIdx.y * 1024 + threadIdx.x, step = (long)gridDim.y * 1024;
    if (vec) {
#pragma unroll 4
        for (long i = first; i < n / 8; i += step) {
            Pack16 av, bv;
            av.u = reinterpret_cast<const uint4 *>(a)[i];
            bv.u = reinterpret_cast<const uint4 *>(b)[i];
#pragma unroll
            for (int e = 0; e < 8; ++e) add(av.h[e], bv.h[e]);
        }
    } else {
        for (long i = first; i < n; i += step) add(a[i], b[i]);
    }
    sd = wave_sum(sd);
    sr = wave_sum(sr);
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = sd;
        part[1][threadIdx.x >> 6] = sr;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double td = 0.0, tr = 0.0;
        for (int w = 0; w < 16; ++w) {
            td += part[0][w];
            tr += part[1][w];
        }
        if (part_out) {
            double *o = part_out + 2 * ((size_t)blockIdx.x * gridDim.y + blockIdx.y);
            o[0] = td;
            o[1] = tr;
        } else {
            diff_norm[blockIdx.x] = sqrt(td);
            ref_norm[blockIdx.x] = sqrt(tr);
        }
    }
}
__global__ __launch_bounds__(64) void deviation_finish_kernel(const double *__restrict__ part,
                                                               double *__restrict__ diff_norm,
                                                               double *__restrict__ ref_norm)
{
    const double *p = part + 2 * ((size_t)blockIdx.x * DEV_PARTS + threadIdx.x);
    const double td = wave_sum(p[0]), tr = wave_sum(p[1]);
    if (threadIdx.x == 0) {
        diff_norm[blockIdx.x] = sqrt(td);
        ref_norm[blockIdx.x] = sqrt(tr);
    }
}
// part: B * DEV_PARTS * 2 doubles, or null for callers without scratch memory
int deviation(const f16 *xq, const f16 *x, int B, long n, double *part, double *diff_norm, double *ref_norm, hipStream_t st)
{
    const int vec = n % 8 == 0 && ((reinterpret_cast<uintptr_t>(xq) | reinterpret_cast<uintptr_t>(x)) & 15) == 0;
    deviation_kernel<<<dim3(B, part ? DEV_PARTS : 1), dim3(1024), 0, st>>>(xq, x, n, vec, part, diff_norm, ref_norm);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    if (part) deviation_finish_kernel<<<dim3(B), dim3(64), 0, st>>>(part, diff_norm, ref_norm);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

inline size_t up256(size_t n) { return (n + 255) & ~(size_t)255; }

template <typename EPI = FpPlain>
int fp_gemm(const f16 *x, int M, int K, const void *W, int N, const f16 *residual, f16 *y, hipStream_t st, const EPI &epi = {})
{
    const auto launch = [&](auto kernel, int bm, int bn) {
        const int tiles_m = (M + bm - 1) / bm, tiles_n = (N + bn - 1) / bn;
        kernel<<<dim3(tiles_m * tiles_n), dim3(512), 0, st>>>(x, M, K, (const f16 *)W, N, residual, y, tiles_m, tiles_n, epi);
    };
    // By rounds of 256 workgroups, in us for 4096 channels (measured over 64 to 2560 rows, 4096 to 22016 columns and both
    // depths of a 7B block: a round of the smaller tiles is shorter by less than they are smaller)
    const auto rounds = [&](int bm, int bn) {
        return (int)(((long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) + 255) / 256);
    };
    const int t64 = 30 * rounds(64, 128), t128 = 38 * rounds(128, 128), t256 = 57 * rounds(128, 256), t512 = 108 * rounds(256, 256),
              t640 = 118 * rounds(320, 256);
    // (320 x 256 is no faster a tile, but where its rounds are fewer a launch is: 1280 x 15360 x 5120 on 240 workgroups 177 us, 262 on 300 of 256 x 256,
    // 1280 x 27648 x 5120 337, 444)
    if (t640 < min(min(t64, t128), min(t256, t512))) launch(fp_gemm_kernel<2, 4, 5, 2, 2, 1, EPI>, 320, 256);
    else if (t64 <= min(min(t128, t256), t512)) launch(fp_gemm_kernel<2, 4, 1, 1, 6, 3, EPI>, 64, 128);
    else if (t128 <= min(t256, t512)) launch(fp_gemm_kernel<2, 4, 2, 1, 4, 3, EPI>, 128, 128);
    else if (t256 <= t512) launch(fp_gemm_kernel<2, 4, 2, 2, 3, 3, EPI>, 128, 256);
    else launch(fp_gemm_kernel<2, 4, 4, 2, 2, 1, EPI>, 256, 256);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

int check_fp_layer(const quota_fp_layer *L, int B, int N)
{
    if (!L) return QUOTA_ERR_NULL;
    if (!L->gamma1 || !L->gamma2 || !L->cosT || !L->sinT || !L->wqkv || !L->wo || !L->wgu || !L->wdown)
        return QUOTA_ERR_NULL;
    if (B <= 0 || N <= 0 || L->H <= 0 || L->F <= 0 || L->n_pos <= 0 || !(L->eps >= 0.0f)) return QUOTA_ERR_INVALID_ARG;
    const int Hkv = L->Hkv > 0 ? L->Hkv : L->H;
    if ((L->dh != 64 && L->dh != 128) || L->H % Hkv != 0 || L->F % 32 != 0) return QUOTA_ERR_SHAPE;
    if (!on_lds_copies(L->wqkv) || !on_lds_copies(L->wo) || !on_lds_copies(L->wgu) || !on_lds_copies(L->wdown))
        return QUOTA_ERR_INVALID_ARG;
    return QUOTA_OK;
}

struct FpWs {
    f16 *h, *q, *k, *v, *o, *x1, *z;
    void *attn;
    size_t bytes;
};

FpWs carve_fp(void *ws, const quota_fp_layer *L, int B, int N)
{
    const int Hkv = L->Hkv > 0 ? L->Hkv : L->H;
    const size_t M = (size_t)B * N, d = (size_t)L->H * L->dh, dkv = (size_t)Hkv * L->dh, F = L->F;
    char *const start = quota_ws_start(ws), *p = start;
    FpWs w;
    auto take = [&](size_t bytes) { void *r = p; p += up256(bytes); return r; };
    w.h = (f16 *)take(M * d * 2);
    w.q = (f16 *)take(M * d * 2);
    w.k = (f16 *)take(M * dkv * 2);
    w.v = (f16 *)take(M * dkv * 2);
    w.o = (f16 *)take(M * d * 2);
    w.x1 = (f16 *)take(M * d * 2);
    w.z = (f16 *)take(M * F * 2);
    w.attn = take(quota_attention_workspace_bytes(B, N, L->H, L->dh));
    w.bytes = (size_t)(p - start) + QUOTA_WS_SLACK;
    return w;
}

}  // namespace

extern "C" size_t quota_fp_block_workspace_bytes(const quota_fp_layer *L, int B, int N)
{
    if (check_fp_layer(L, B, N) != QUOTA_OK) return 0;
    return carve_fp(nullptr, L, B, N).bytes;
}

extern "C" int quota_fp_block(const quota_fp_layer *L, const void *x_f16, const int32_t *pos, int B, int N,
                              void *x_out_f16, void *ws, void *stream)
{
    int rc = check_fp_layer(L, B, N);
    if (rc != QUOTA_OK) return rc;
    if (!x_f16 || !pos || !x_out_f16 || !ws) return QUOTA_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    const int H = L->H, dh = L->dh, F = L->F, Hkv = L->Hkv > 0 ? L->Hkv : H, d = H * dh, dkv = Hkv * dh;
    const int M = B * N;
    const f16 *x = (const f16 *)x_f16;
    FpWs w = carve_fp(ws, L, B, N);

    fp_rmsnorm_kernel<<<dim3(M), dim3(256), 0, st>>>(x, d, L->gamma1, L->eps, w.h);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    const FpRope rope = {pos, L->cosT, L->sinT, L->n_pos, d, dkv, dh, w.q, w.k, w.v};
    if ((rc = fp_gemm(w.h, M, d, L->wqkv, d + 2 * dkv, nullptr, nullptr, st, rope)) != QUOTA_OK) return rc;
    if ((rc = quota_attention_prefill_gqa(w.q, w.k, w.v, B, N, H, Hkv, dh, 0, 0, w.o, nullptr, nullptr, w.attn,
                                          stream)) != QUOTA_OK)
        return rc;
    if ((rc = fp_gemm(w.o, M, d, L->wo, d, x, w.x1, st)) != QUOTA_OK) return rc;
    fp_rmsnorm_kernel<<<dim3(M), dim3(256), 0, st>>>(w.x1, d, L->gamma2, L->eps, w.h);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    if ((rc = fp_gemm(w.h, M, d, L->wgu, 2 * F, nullptr, w.z, st, FpSilu{})) != QUOTA_OK) return rc;
    return fp_gemm(w.z, M, F, L->wdown, d, w.x1, (f16 *)x_out_f16, st);
}

extern "C" int quota_activation_deviation(const void *xq_f16, const void *x_f16, int B, long n_per_sample,
                                          double *diff_norm, double *ref_norm, void *stream)
{
    if (!xq_f16 || !x_f16 || !diff_norm || !ref_norm) return QUOTA_ERR_NULL;
    if (B <= 0 || n_per_sample < 0) return QUOTA_ERR_INVALID_ARG;
    return deviation((const f16 *)xq_f16, (const f16 *)x_f16, B, n_per_sample, nullptr, diff_norm, ref_norm,
                     (hipStream_t)stream);
}

namespace {
struct ProfileWs {
    f16 *xq, *xf;
    int32_t *pos_out;
    double *part;
    void *rest;
    size_t bytes;
};
ProfileWs carve_profile(void *ws, const quota_layer *Lq, const quota_fp_layer *Lf, int B, int N)
{
    const size_t M = (size_t)B * N, d = (size_t)Lf->H * Lf->dh;
    char *const start = quota_ws_start(ws), *p = start;
    ProfileWs w;
    auto take = [&](size_t bytes) { void *r = p; p += up256(bytes); return r; };
    w.xq = (f16 *)take(M * d * 2);
    w.xf = (f16 *)take(M * d * 2);
    w.pos_out = (int32_t *)take(M * 4);
    w.part = (double *)take((size_t)B * DEV_PARTS * 2 * sizeof(double));
    const size_t a = quota_prefill_workspace_bytes(Lq, B, N), b = quota_fp_block_workspace_bytes(Lf, B, N);
    w.rest = take(a > b ? a : b);           // the two runs are ordered on one stream and share it
    w.bytes = (size_t)(p - start) + QUOTA_WS_SLACK;
    return w;
}
}  // namespace

extern "C" size_t quota_profile_block_workspace_bytes(const quota_layer *Lq, const quota_fp_layer *Lf, int B,
                                                      int N)
{
    if (!Lq || check_fp_layer(Lf, B, N) != QUOTA_OK) return 0;
    return carve_profile(nullptr, Lq, Lf, B, N).bytes;
}

extern "C" int quota_profile_block(const quota_layer *Lq, const quota_fp_layer *Lf, const void *x_f16,
                                   const int32_t *pos, int B, int N, quota_kv_cache *scratch_cache,
                                   double *diff_norm, double *ref_norm, void *ws, void *stream)
{
    if (!Lq || !Lf || !x_f16 || !pos || !scratch_cache || !diff_norm || !ref_norm || !ws) return QUOTA_ERR_NULL;
    int rc = check_fp_layer(Lf, B, N);
    if (rc != QUOTA_OK) return rc;
    const int Hkv_q = Lq->Hkv > 0 ? Lq->Hkv : Lq->H, Hkv_f = Lf->Hkv > 0 ? Lf->Hkv : Lf->H;
    if (Lq->H != Lf->H || Lq->dh != Lf->dh || Lq->F != Lf->F || Hkv_q != Hkv_f) return QUOTA_ERR_SHAPE;
    ProfileWs w = carve_profile(ws, Lq, Lf, B, N);

    // the deployed low-bit block, nothing pruned; it validates its own arguments before any launch
    quota_state s;
    s.B = B; s.N = N; s.vis_begin = 0; s.Nv = 0;
    s.x = x_f16; s.pos = pos; s.x_out = w.xq; s.pos_out = w.pos_out;
    quota_score_params p;
    quota_score_params_default(&p);
    const int len0 = scratch_cache->len;
    rc = quota_prefill_layer(Lq, &s, QUOTA_KEEP_ALL, &p, scratch_cache, nullptr, w.rest, stream);
    scratch_cache->len = len0;              // the rows written are scratch: the cache is handed back as it came
    if (rc != QUOTA_OK) return rc;
    if ((rc = quota_fp_block(Lf, x_f16, pos, B, N, w.xf, w.rest, stream)) != QUOTA_OK) return rc;
    return deviation(w.xq, w.xf, B, (long)N * Lf->H * Lf->dh, w.part, diff_norm, ref_norm, (hipStream_t)stream);
}
