// Quantizers of the W4A4 execution form: weight group quantizer + repack,
// per-token int4 activation quantizer (the Q of Eq. 6) and its fused variants
// (RMSNorm in front of QKV / gate-up, SwiGLU product in front of down).
// All are row kernels: in launches of 2048 rows and more of up to 6144 columns one wave per row
// (four rows per workgroup), else one workgroup per row; the row is cached in registers as
// 16-byte chunks, absmax / sums of squares are wave or block reductions, 8 codes are stored per
// chunk: a packed dword, or 6 bytes of e2m3 numbers for the GEMM.  HBM-bound by design.
#include <type_traits>

#include "common.h"
#include "internal.h"
#include "rowquant.h"

// ------------------------------------------------------------ W4 weights

// one wave per (row n, group g): 2 elements per lane
__global__ __launch_bounds__(256) void quantize_weights_kernel(
    const float *__restrict__ w, int N, int K, int G, int8_t *__restrict__ codes,
    f16 *__restrict__ scales)
{
    long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    if (wave >= (long)N * G) return;
    int n = (int)(wave / G), g = (int)(wave % G);
    int k = g * QUOTA_GROUP_W + 2 * lane;
    const float *wr = w + (size_t)n * K;
    float v0 = k < K ? wr[k] : 0.0f;
    float v1 = k + 1 < K ? wr[k + 1] : 0.0f;
    float a = wave_max(fmaxf(fabsf(v0), fabsf(v1)));
    f16 sh = to_f16(a / 7.0f);
    float s = (float)sh;
    if (a == 0.0f || s == 0.0f) { sh = (f16)1.0f; s = 1.0f; }
    if (lane == 0) scales[(size_t)n * G + g] = sh;
    if (k < K) codes[(size_t)n * K + k] = (int8_t)code_from(rintf(v0 / s));
    if (k + 1 < K) codes[(size_t)n * K + k + 1] = (int8_t)code_from(rintf(v1 / s));
}

// The same for rows of whole 8-channel chunks: a thread owns chunks of 8 channels (two 16-byte loads,
// one 8-byte store), the 16 chunks of a group are 16 neighbouring lanes that share their absmax by row
// rotations.  Four chunks per thread are loaded before the first is used: bound by HBM (5 bytes per
// weight); 22016 x 4096: 159 us with 2 channels per lane and one load in flight.
constexpr int QW_UN = 4;
__device__ __forceinline__ float row16_max(float a)
{
#define STEP(ctrl)                                                                                        \
    a = fmaxf(a, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(a), __float_as_int(a), ctrl, 0xf, 0xf, false)))
    STEP(0x121); STEP(0x122); STEP(0x124); STEP(0x128);            // rotations of a row of 16 lanes
#undef STEP
    return a;
}
__global__ __launch_bounds__(256) void quantize_weights8_kernel(
    const float *__restrict__ w, int K, int G, long total, int8_t *__restrict__ codes,
    f16 *__restrict__ scales)
{
    float v[QW_UN][8];
    long item[QW_UN];
#pragma unroll
    for (int u = 0; u < QW_UN; ++u) {
        item[u] = ((long)blockIdx.x * QW_UN + u) * 256 + threadIdx.x;         // (row, group, chunk) in order
        const long ng = min(item[u], total - 1) >> 4;
        const int n = (int)(ng / G), k = (int)(ng % G) * QUOTA_GROUP_W + 8 * (threadIdx.x & 15);
        const float4 *src = reinterpret_cast<const float4 *>(w + (size_t)n * K + min(k, K - 8));
        *reinterpret_cast<float4 *>(v[u]) = src[0];
        *reinterpret_cast<float4 *>(v[u] + 4) = src[1];
    }
#pragma unroll
    for (int u = 0; u < QW_UN; ++u) {
        const long ng = item[u] >> 4;
        const int n = (int)(ng / G), g = (int)(ng % G), k = g * QUOTA_GROUP_W + 8 * (threadIdx.x & 15);
        float a = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(v[u][e]));      // (a clamped chunk repeats one of the group's)
        a = row16_max(a);
        f16 sh = to_f16(a / 7.0f);
        float s = (float)sh;
        if (a == 0.0f || s == 0.0f) { sh = (f16)1.0f; s = 1.0f; }
        if (item[u] >= total) continue;
        if ((threadIdx.x & 15) == 0) scales[ng] = sh;
        if (k < K) {
            uint32_t o[2] = {0, 0};
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e >> 2] |= (uint32_t)(uint8_t)(int8_t)code_from(rintf(v[u][e] / s)) << (8 * (e & 3));
            *reinterpret_cast<uint2 *>(codes + (size_t)n * K + k) = make_uint2(o[0], o[1]);
        }
    }
}

// Quantizer and repack in one pass: a thread owns the same chunk of four neighbouring rows, so that what a
// workgroup writes for a group is 256 bytes in one piece of the [G][N] layout.  Bound by HBM (4.5 bytes per
// weight); 22016 x 4096: the two separate passes take 84 + 25 us and move 590 MB, this one 79 us and 409 MB.
__global__ __launch_bounds__(256) void quantize_pack_weights_kernel(
    const float *__restrict__ w, int N, int K, int G, long total, uint32_t *__restrict__ packed,
    f16 *__restrict__ scales_t)
{
    const long item = (long)blockIdx.x * 256 + threadIdx.x;         // (four rows, group, chunk) in order
    const long ng = min(item, total - 1) >> 4;
    const int n = 4 * (int)(ng / G), g = (int)(ng % G), chunk = threadIdx.x & 15, k = g * QUOTA_GROUP_W + 8 * chunk;
    float v[4][8];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float4 *src = reinterpret_cast<const float4 *>(w + (size_t)(n + u) * K + min(k, K - 8));
        *reinterpret_cast<float4 *>(v[u]) = src[0];
        *reinterpret_cast<float4 *>(v[u] + 4) = src[1];
    }
    union { uint2 u; f16 h[4]; } sh;
    uint32_t word[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        float a = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf(v[u][e]));      // (a clamped chunk repeats one of the group's)
        a = row16_max(a);
        f16 h = to_f16(a / 7.0f);
        float s = (float)h;
        if (a == 0.0f || s == 0.0f) { h = (f16)1.0f; s = 1.0f; }
        sh.h[u] = h;
        word[u] = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) word[u] |= ((uint32_t)code_from(rintf(v[u][e] / s)) & 0xFu) << (4 * e);
    }
    if (item >= total) return;
    const size_t at = (size_t)g * N + n;
#pragma unroll
    for (int u = 0; u < 4; ++u) packed[(at + u) * 16 + chunk] = k < K ? word[u] : 0u;
    if (chunk == 0) *reinterpret_cast<uint2 *>(scales_t + at) = sh.u;
}

// four int8 codes (bytes) -> four nibbles in the low half
__device__ __forceinline__ uint32_t nibbles4(uint32_t b)
{
    b &= 0x0F0F0F0Fu;
    b |= b >> 4;                                    // nibble pairs in bytes 0 and 2
    return (b & 0xFFu) | ((b >> 8) & 0xFF00u);
}

// The repack for aligned codes: a thread turns 32 codes (two 16-byte loads, K is a multiple of 32) into
// the 16-byte piece number t % 4 of row n in group g.
__global__ __launch_bounds__(256) void pack_weights16_kernel(
    const int8_t *__restrict__ codes, const f16 *__restrict__ scales, int N, int K, int G,
    uint4 *__restrict__ packed, f16 *__restrict__ scales_t)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= (long)G * N * 4) return;
    const int i = (int)(t & 3);
    const long gn = t >> 2;
    const int n = (int)(gn % N), g = (int)(gn / N), k = g * QUOTA_GROUP_W + 32 * i;
    uint4 o = make_uint4(0, 0, 0, 0);
    if (k < K) {
        const uint4 *src = reinterpret_cast<const uint4 *>(codes + (size_t)n * K + k);
        const uint4 a = src[0], b = src[1];
        o.x = nibbles4(a.x) | nibbles4(a.y) << 16;
        o.y = nibbles4(a.z) | nibbles4(a.w) << 16;
        o.z = nibbles4(b.x) | nibbles4(b.y) << 16;
        o.w = nibbles4(b.z) | nibbles4(b.w) << 16;
    }
    packed[t] = o;
    if (i == 0) scales_t[(size_t)g * N + n] = scales[(size_t)n * G + g];
}

// codes int8 [N][K] -> packed [G][N][16 dwords]; scales [N][G] -> [G][N]
__global__ __launch_bounds__(256) void pack_weights_kernel(
    const int8_t *__restrict__ codes, const f16 *__restrict__ scales, int N, int K, int G,
    uint32_t *__restrict__ packed, f16 *__restrict__ scales_t)
{
    long t = (long)blockIdx.x * 256 + threadIdx.x;
    long total = (long)G * N * 16;
    if (t >= total) return;
    int i = (int)(t & 15);
    long gn = t >> 4;
    int n = (int)(gn % N), g = (int)(gn / N);
    int k0 = g * QUOTA_GROUP_W + 8 * i;
    uint32_t word = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        int k = k0 + e;
        int c = k < K ? (int)codes[(size_t)n * K + k] : 0;
        word |= (uint32_t)(c & 0xF) << (4 * e);
    }
    packed[t] = word;
    if (i == 0) scales_t[(size_t)g * N + n] = scales[(size_t)n * G + g];
}

// ------------------------------------------------- activation quantizers

// A row is owned by GROUP threads, each caching NCH chunks (2 to 16).  Every load of a thread is
// issued before the first use (unconditional loads at clamped indices instead of guarded ones, so
// that nothing separates them): one memory round trip per kernel.  GROUP = 64 (rows of up to 6144
// columns): one WAVE per row, four rows per workgroup -- a lane issues all its 16-byte loads back
// to back, the reductions are wave shuffles and there is no workgroup barrier.  GROUP = 256 or 512 (up to
// 32768 columns): the whole workgroup owns the row and reduces through LDS.
// Below this many rows the launch cannot fill the chip with one wave per row, and a row is
// finished sooner by a whole workgroup (512 threads for a layer's few wide rows: with_row_shape).
#define ROW_WAVE_MIN_ROWS 2048

constexpr int row_threads(int group) { return group == 64 ? 256 : group; }
template <int GROUP, bool MAX, bool SUM, bool FRESH = false>
__device__ __forceinline__ void group_reduce(float &mx, double &sum, double *sm)
{
    if (GROUP == 64) {
        if (MAX) mx = wave_absmax(mx);
        if (SUM) sum = wave_sum(sum);
    } else {
        block_max_sum<GROUP / 64, MAX, SUM, FRESH>(mx, sum, sm);
    }
}
// A launch's arguments that are not in registers when a wave starts (structures and what is behind them) come from memory, the first touch of
// each 64 bytes from far away.  Left alone the compiler asks for them where they are used, in the middle of a row's chain: they are wanted
// here, where the row's loads are on their way.  (Read, not replaced: of a pointer that comes out of assembly the compiler does not know that its
// memory is global, and stores through it are flat ones, which take the LDS's path too: 3 x 18944 3.31 us, 3.04 so, 32 x 13824 3.06, 2.78, 640 x 11008 7.85, 7.33.)
template <typename ARG>
__device__ __forceinline__ void argument_now(const ARG &a) { asm volatile("" ::"s"(a)); }
template <int GROUP, typename OUT, typename... ARGS>
__device__ __forceinline__ void row_arguments_now(const OUT &q, const ARGS &...args)
{
    if constexpr (GROUP != 64) {                         // (long launches take what registers there are)
        argument_now(q.q);
        if constexpr (OUT::STARTS) argument_now(q.rows);
        (argument_now(args), ...);
    }
}
#define ROW_PROLOGUE()                                                                         \
    __shared__ __align__(16) double sm[GROUP == 64 ? 2 : 6 * GROUP / 64];                                                  \
    const int lane = threadIdx.x % GROUP;                                                      \
    const int row = row_wg<OUT>(blockIdx.x, (M + row_threads(GROUP) / GROUP - 1) / (row_threads(GROUP) / GROUP)) * (row_threads(GROUP) / GROUP) + (GROUP == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / GROUP) : 0); \
    if (row >= M) return;     /* GROUP = 64: the whole wave leaves; else never taken */ \
    (void)sm

template <bool WANT_METRICS, int GROUP, int NCH, typename OUT>
__global__ __launch_bounds__(row_threads(GROUP)) void quantize_act_kernel(
    const f16 *__restrict__ x, int M, int d, long ldx, int rows_per_seq, long seq_stride,
    OUT q, float *__restrict__ scale, float *__restrict__ sumsq,
    float *__restrict__ ressq)
{
    ROW_PROLOGUE();
    const int nchunk = d >> 3;
    const bool first = row < rows_per_seq;               // (all rows of a dense tensor: no division)
    const uint4 *xr = reinterpret_cast<const uint4 *>(
        x + (first ? (size_t)row * ldx : (size_t)(row / rows_per_seq) * seq_stride + (size_t)(row % rows_per_seq) * ldx));
    Pack16 v[NCH];
    float a = 0.0f;
    double ss = 0.0;
#pragma unroll
    for (int r = 0; r < NCH; ++r) v[r].u = xr[min(lane + GROUP * r, nchunk - 1)];
    row_arguments_now<GROUP>(q, scale);
    if constexpr (WANT_METRICS) row_arguments_now<GROUP>(q, sumsq, ressq);
    RowStore<OUT> store;
    if (GROUP != 64) store.make(lane, row);
    const OUT to = row_out(q, row, nchunk);
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        int c = lane + GROUP * r;
        if (c < nchunk) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = (float)v[r].h[e];
                a = fmaxf(a, fabsf(f));
                if (WANT_METRICS) ss = __builtin_fma((double)f, (double)f, ss);     // product exact in fp64
            }
        }
    }
    group_reduce<GROUP, true, WANT_METRICS, true>(a, ss, sm);
    float s;
    if (GROUP == 64) store.make(lane, row);
    double rs = quantize_cached_row<WANT_METRICS, GROUP, NCH>(v, nchunk, lane, a, to, store, s);
    if (WANT_METRICS) { float dummy = 0.0f; group_reduce<GROUP, false, true>(dummy, rs, sm); }
    if (lane == 0) {
        if (scale) scale[row] = s;
        if (WANT_METRICS) {
            if (sumsq) sumsq[row] = (float)ss;
            if (ressq) ressq[row] = (float)rs;
        }
    }
}

// Workgroups behind the quantizer's, one per kept row (see quota_kept_copies; the gather of kv.hip has such copies among the loads and stores of the row
// that it quantizes)
struct NoCopies {};
template <int THREADS>
__device__ __forceinline__ void copy_kept_row(const quota_kept_copies &c, int m)
{
    const int b = m / c.kept.n_keep, j = m - b * c.kept.n_keep, src = c.kept.row(j, c.kept.index(b, j));
    const size_t from = (size_t)b * c.kept.N + src, to = (size_t)b * c.capacity + c.len + j;
    const int nkv = c.dkv >> 3, ng = c.dkv >> 6;         // dwords of codes, group scales per K or V row
    for (int i = threadIdx.x; i < nkv; i += THREADS) {
        const uint32_t k = c.skc[from * nkv + i], v = c.svc[from * nkv + i];
        c.ckc[to * nkv + i] = k;
        c.cvc[to * nkv + i] = v;
    }
    if ((int)threadIdx.x < ng) {
        c.cks[to * ng + threadIdx.x] = c.sks[from * ng + threadIdx.x];
        c.cvs[to * ng + threadIdx.x] = c.svs[from * ng + threadIdx.x];
    }
    if (threadIdx.x == 0) {
        c.pos_out[m] = c.pos[from];
        c.rows_out[m] = src;
    }
}

template <bool WANT_METRICS, int GROUP, int NCH, typename OUT, typename COPIES = NoCopies>
__global__ __launch_bounds__(row_threads(GROUP)) void rmsnorm_quantize_act_kernel(
    const f16 *__restrict__ x, int M, int d, long ldx, const float *__restrict__ gamma, float eps,
    OUT q, float *__restrict__ scale, float *__restrict__ sumsq,
    float *__restrict__ ressq, f16 *__restrict__ h_out, COPIES copies)
{
    if constexpr (!std::is_same_v<COPIES, NoCopies>) {
        if ((int)blockIdx.x >= M) {
            copy_kept_row<row_threads(GROUP)>(copies, blockIdx.x - M);
            return;
        }
    }
    ROW_PROLOGUE();
    const int nchunk = d >> 3;
    const uint4 *xr = reinterpret_cast<const uint4 *>(x + (size_t)row * ldx);
    Pack16 v[NCH];
    float a_raw = 0.0f;
    double ss = 0.0;
    // wave-per-row launches are long (thousands of rows): the gains are fetched where they are used
    // (they stay in cache) so that more waves fit on a SIMD; workgroup-per-row launches are short and
    // latency counts, so there every load is issued up front
    constexpr bool GAINS_EARLY = GROUP != 64;
    float4 ga[GAINS_EARLY ? NCH : 1][2];
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        const int c = min(lane + GROUP * r, nchunk - 1);
        v[r].u = xr[c];
        if (GAINS_EARLY) {
            const float4 *gp = reinterpret_cast<const float4 *>(gamma + 8 * c);
            ga[r][0] = gp[0];
            ga[r][1] = gp[1];
        }
    }
    row_arguments_now<GROUP>(q, scale, h_out);
    if constexpr (WANT_METRICS) row_arguments_now<GROUP>(q, sumsq, ressq);
    RowStore<OUT> store;
    if (GROUP != 64) store.make(lane, row);
    const OUT to = row_out(q, row, nchunk);
    double per_channel = 1.0 / (double)d;
    if (GROUP != 64) {
        asm volatile("" : "+v"(per_channel));
        __builtin_amdgcn_sched_barrier(0);               // (here, while the row is on its way)
    }
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        int c = lane + GROUP * r;
        if (c < nchunk) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = (float)v[r].h[e];
                a_raw = fmaxf(a_raw, fabsf(f));
                ss = __builtin_fma((double)f, (double)f, ss);     // product exact in fp64
            }
        }
    }
    group_reduce<GROUP, WANT_METRICS, true, true>(a_raw, ss, sm);
    if (!GAINS_EARLY) {
        // the row stays packed (32 registers for 4096 columns): without this the compiler keeps the 64
        // converted floats of the first pass alive for the second one
#pragma unroll
        for (int r = 0; r < NCH; ++r)
            asm volatile("" : "+v"(v[r].u.x), "+v"(v[r].u.y), "+v"(v[r].u.z), "+v"(v[r].u.w));
    }
    const float rn = inv_sqrt(ss * per_channel + (double)eps);
    float s_raw = 1.0f, inv_raw = 0.0f;
    if (a_raw != 0.0f) { s_raw = a_raw / 7.0f; inv_raw = 7.0f / a_raw; }
    float a = 0.0f;
    double rs = 0.0;
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        int c = lane + GROUP * r;
        if (c < nchunk) {
            const float4 *gp = reinterpret_cast<const float4 *>(gamma + 8 * c);
            const float4 g0 = GAINS_EARLY ? ga[GAINS_EARLY ? r : 0][0] : gp[0];
            const float4 g1 = GAINS_EARLY ? ga[GAINS_EARLY ? r : 0][1] : gp[1];
            float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = (float)v[r].h[e];
                if (WANT_METRICS) {
                    float deq = code_float(code_bits(f * inv_raw)) * s_raw;
                    float rr = deq - f;
                    rs = __builtin_fma((double)rr, (double)rr, rs);
                }
                float hn = f * rn;
                hn = hn * gm[e];
                f16 hh = to_f16(hn);
                v[r].h[e] = hh;
                a = fmaxf(a, fabsf((float)hh));
            }
            if (h_out) reinterpret_cast<uint4 *>(h_out + (size_t)row * d)[c] = v[r].u;
        }
        // keep the compiler from hoisting every chunk's gain loads to the top (that costs 64 registers)
        if (!GAINS_EARLY) __builtin_amdgcn_sched_barrier(0);
    }
    group_reduce<GROUP, true, WANT_METRICS, !WANT_METRICS>(a, rs, sm);
    float s;
    if (GROUP == 64) store.make(lane, row);
    quantize_cached_row<false, GROUP, NCH>(v, nchunk, lane, a, to, store, s);
    if (lane == 0) {
        scale[row] = s;
        if (WANT_METRICS) {
            if (sumsq) sumsq[row] = (float)ss;
            if (ressq) ressq[row] = (float)rs;
        }
    }
}

// EARLY: every load before the first use (short launches, latency counts); otherwise chunk by
// chunk (long launches: fewer live registers, more waves per SIMD to hide the latency instead).
template <int GROUP, int NCH, bool EARLY, typename OUT>
__global__ __launch_bounds__(row_threads(GROUP)) void silu_mul_quantize_act_kernel(
    const f16 *__restrict__ gu, int M, int F, OUT q, float *__restrict__ scale,
    f16 *__restrict__ z_out, const f16 *__restrict__ z_inject)
{
    ROW_PROLOGUE();
    const int nchunk = F >> 3;
    const uint4 *gr = reinterpret_cast<const uint4 *>(gu + (size_t)row * 2 * F);
    const uint4 *ur = reinterpret_cast<const uint4 *>(gu + (size_t)row * 2 * F + F);
    Pack16 v[NCH], gg[NCH], uu[NCH];
    float a = 0.0f;
    if (z_inject) {
#pragma unroll
        for (int r = 0; r < NCH; ++r)
            v[r].u = reinterpret_cast<const uint4 *>(z_inject + (size_t)row * F)[min(lane + GROUP * r, nchunk - 1)];
    } else if (EARLY) {
#pragma unroll
        for (int r = 0; r < NCH; ++r) {
            const int c = min(lane + GROUP * r, nchunk - 1);
            gg[r].u = gr[c];
            uu[r].u = ur[c];
        }
    }
    row_arguments_now<GROUP>(q, scale, z_out);
    RowStore<OUT> store;
    if (GROUP != 64) store.make(lane, row);
    const OUT to = row_out(q, row, nchunk);
#pragma unroll
    for (int r = 0; r < NCH; ++r) {
        int c = lane + GROUP * r;
        if (c < nchunk) {
            if (!z_inject) {
                if (!EARLY) { gg[r].u = gr[c]; uu[r].u = ur[c]; }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[r].h[e] = silu_mul((float)gg[r].h[e], (float)uu[r].h[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf((float)v[r].h[e]));
            if (z_out) reinterpret_cast<uint4 *>(z_out + (size_t)row * F)[c] = v[r].u;
        }
    }
    double none = 0.0;
    group_reduce<GROUP, true, false, true>(a, none, sm);
    float s;
    if (GROUP == 64) store.make(lane, row);
    quantize_cached_row<false, GROUP, NCH>(v, nchunk, lane, a, to, store, s);
    if (lane == 0) scale[row] = s;
}

// ------------------------------------------------------------ host side

// Calls launch(GROUP, NCH, grid) with the smallest cache that holds d columns: a thread's registers are what limits the
// rows in flight.  RMSNorm quantizer with metrics, 11776 rows of 5120 columns: 61 us with 12 chunks per lane, of which 10
// are used, 113 with 8 per thread of a workgroup, of which 2.5 are used.  MOST: the most columns that the caller lets by.
template <typename OUT, int MOST = ROW_MAXCOLS, typename LAUNCH>
static void with_row_shape(int M, int d, LAUNCH launch)
{
    const auto go = [&](auto group, auto nch) { launch(group, nch, dim3(group() == 64 ? (M + 3) / 4 : M)); };
    const std::integral_constant<int, 64> wave;
    const std::integral_constant<int, 256> workgroup;
    if constexpr (OUT::MANY) {
        if (M >= ROW_WAVE_MIN_ROWS && d <= 64 * 8 * 12) {
            if (d <= 64 * 8 * 2) go(wave, std::integral_constant<int, 2>());
            else if (d <= 64 * 8 * 8) go(wave, std::integral_constant<int, 8>());
            else go(wave, std::integral_constant<int, 12>());
            return;
        }
    }
    // A layer's few rows, wider than 2048 columns, by 512 threads each: one wave a SIMD waits between its instructions.  (16 x 4096 and 16 x 11008 of a decode
    // step of 16 sequences over 32 layers, 1904 -> 1885 us; 32 layers of 640 to 122 rows 4158 -> 4137, one of 165 rows 109.7 -> 109.0; 1024 threads 1907, 4161 and 109.5;
    // 16 layers of 512 channels take 0.5 % longer with 512.)  The plain quantizers gain most: with 256 threads and 512, us, 16 x 4096 2.30, 2.05, 16 x 11008 3.64, 2.63, 32 x
    // 13824 4.00, 2.77, 165 x 11008 4.51, 3.60, 500 x 11008 6.55, 5.65, with the SiLU product 165 x 11008 5.62, 5.03; with RMSNorm 16 x 4096 2.56, 2.41, 165 x 4096 3.00, 2.81,
    // 300 and 500 x 4096 as long; all of them so a 16-sequence step 1793, 1750 and the batch-1 stack 4001, 3972.
    if constexpr (!OUT::MANY) {
        const std::integral_constant<int, 512> wide;
        if (d <= 2048) go(workgroup, std::integral_constant<int, 2>());
        else if (d <= 512 * 8) go(wide, std::integral_constant<int, 1>());
        else if (d <= 512 * 8 * 2) go(wide, std::integral_constant<int, 2>());
        else if (d <= 512 * 8 * 4) go(wide, std::integral_constant<int, 4>());
        else if constexpr (MOST > 512 * 8 * 4) go(wide, std::integral_constant<int, 8>());
    } else {
        if (d <= 256 * 8 * 2) go(workgroup, std::integral_constant<int, 2>());
        else if (d <= 256 * 8 * 4) go(workgroup, std::integral_constant<int, 4>());
        else if (d <= 256 * 8 * 8) go(workgroup, std::integral_constant<int, 8>());
        else if constexpr (MOST > 256 * 8 * 8) go(workgroup, std::integral_constant<int, 16>());
    }
}

extern "C" size_t quota_weights_packed_bytes(int N, int K)
{
    if (N <= 0 || K <= 0) return 0;
    size_t G = ((size_t)K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    return G * (size_t)N * 64;
}

extern "C" size_t quota_weights_scale_bytes(int N, int K)
{
    if (N <= 0 || K <= 0) return 0;
    size_t G = ((size_t)K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    return G * (size_t)N * 2;
}

extern "C" int quota_quantize_weights(const float *w, int N, int K, int8_t *codes,
                                      void *scales_f16, void *stream)
{
    if (!w || !codes || !scales_f16) return QUOTA_ERR_NULL;
    if (N <= 0 || K <= 0) return QUOTA_ERR_INVALID_ARG;
    int G = (K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    long waves = (long)N * G;
    ProfScope prof(QUOTA_K_QUANTIZE_WEIGHTS, 0, 5.0 * N * K + 2.0 * N * G, (hipStream_t)stream);
    if (K % 8 == 0 && (reinterpret_cast<uintptr_t>(w) & 15) == 0 && (reinterpret_cast<uintptr_t>(codes) & 7) == 0)
        quantize_weights8_kernel<<<dim3((unsigned)((16 * waves + 256 * QW_UN - 1) / (256 * QW_UN))), dim3(256), 0,
                                   (hipStream_t)stream>>>(w, K, G, 16 * waves, codes, (f16 *)scales_f16);
    else
        quantize_weights_kernel<<<dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, (hipStream_t)stream>>>(
            w, N, K, G, codes, (f16 *)scales_f16);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

extern "C" int quota_pack_weights(const int8_t *codes, const void *scales_f16,
                                  const quota_weights *W, void *stream)
{
    if (!codes || !scales_f16 || !W || !W->packed || !W->scales) return QUOTA_ERR_NULL;
    if (W->N <= 0 || W->K <= 0) return QUOTA_ERR_INVALID_ARG;
    if (W->N % 64 != 0 || W->K % 32 != 0) return QUOTA_ERR_SHAPE;
    int G = (W->K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    long total = (long)G * W->N * 16;
    ProfScope prof(QUOTA_K_PACK_WEIGHTS, 0, 1.5 * W->N * W->K + 4.0 * W->N * G, (hipStream_t)stream);
    if (((reinterpret_cast<uintptr_t>(codes) | reinterpret_cast<uintptr_t>(W->packed)) & 15) == 0)
        pack_weights16_kernel<<<dim3((unsigned)((total / 4 + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>(
            codes, (const f16 *)scales_f16, W->N, W->K, G, (uint4 *)W->packed, (f16 *)W->scales);
    else
        pack_weights_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>(
            codes, (const f16 *)scales_f16, W->N, W->K, G, (uint32_t *)W->packed, (f16 *)W->scales);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

extern "C" int quota_quantize_pack_weights(const float *w, const quota_weights *W, void *stream)
{
    if (!w || !W || !W->packed || !W->scales) return QUOTA_ERR_NULL;
    if (W->N <= 0 || W->K <= 0) return QUOTA_ERR_INVALID_ARG;
    if (W->N % 64 != 0 || W->K % 32 != 0) return QUOTA_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(w) & 15) || (reinterpret_cast<uintptr_t>(W->packed) & 3) ||
        (reinterpret_cast<uintptr_t>(W->scales) & 7))
        return QUOTA_ERR_INVALID_ARG;
    const int G = (W->K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    const long total = (long)W->N / 4 * G * 16;
    ProfScope prof(QUOTA_K_PACK_WEIGHTS, 0, 4.5 * W->N * W->K + 2.0 * W->N * G, (hipStream_t)stream);
    quantize_pack_weights_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>(
        w, W->N, W->K, G, total, (uint32_t *)W->packed, (f16 *)W->scales);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

static int check_rows(const void *x, int M, int d, int ld, const void *q, const void *scale)
{
    if (!x || !q || !scale) return QUOTA_ERR_NULL;
    if (M < 0 || d <= 0) return QUOTA_ERR_INVALID_ARG;
    if (d % 8 != 0 || d > ROW_MAXCOLS || ld < d || ld % 8 != 0) return QUOTA_ERR_SHAPE;
    return QUOTA_OK;
}

extern "C" int quota_quantize_act(const void *x_f16, int M, int d, int ldx, uint8_t *q_packed,
                                  float *scale, float *sumsq_opt, float *ressq_opt, void *stream)
{
    int rc = check_rows(x_f16, M, d, ldx, q_packed, scale);
    if (rc != QUOTA_OK) return rc;
    if (M == 0) return QUOTA_OK;
    hipStream_t st = (hipStream_t)stream;
    ProfScope prof(QUOTA_K_QUANTIZE_ACT, 0, 2.5 * M * d + 4.0 * M, st);
    with_row_shape<RowOutPacked>(M, d, [&](auto group, auto nch, dim3 grid) {
        auto kernel = sumsq_opt || ressq_opt ? quantize_act_kernel<true, group(), nch(), RowOutPacked>
                                             : quantize_act_kernel<false, group(), nch(), RowOutPacked>;
        kernel<<<grid, dim3(row_threads(group())), 0, st>>>((const f16 *)x_f16, M, d, ldx, M, 0, RowOutPacked{(uint32_t *)q_packed},
                                                   scale, sumsq_opt, ressq_opt);
    });
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

template <typename OUT>
static int rmsnorm_quantize(const void *x_f16, int M, int d, int ldx, const float *gamma, float eps, OUT q,
                            float *scale, float *sumsq_opt, float *ressq_opt, void *h_opt, hipStream_t st)
{
    // a layer's rows have the model's width, and the few of a decode step no metrics
    constexpr bool LAYER = !std::is_same_v<OUT, RowOutPacked>, METRICS = !std::is_same_v<OUT, RowOutFrag>;
    if (LAYER && d > QUOTA_MAX_MODEL_WIDTH) return QUOTA_ERR_SHAPE;
    ProfScope prof(QUOTA_K_RMSNORM_QUANTIZE_ACT, 0, 2.5 * M * d + 4.0 * M + 4.0 * d, st);
    with_row_shape<OUT, LAYER ? QUOTA_MAX_MODEL_WIDTH : ROW_MAXCOLS>(M, d, [&](auto group, auto nch, dim3 grid) {
        auto kernel = rmsnorm_quantize_act_kernel<false, group(), nch(), OUT>;
        if constexpr (METRICS)
            if (sumsq_opt || ressq_opt) kernel = rmsnorm_quantize_act_kernel<true, group(), nch(), OUT>;
        kernel<<<grid, dim3(row_threads(group())), 0, st>>>((const f16 *)x_f16, M, d, ldx, gamma, eps, q, scale, sumsq_opt, ressq_opt,
                                                   (f16 *)h_opt, NoCopies{});
    });
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

extern "C" int quota_rmsnorm_quantize_act(const void *x_f16, int M, int d, int ldx,
                                          const float *gamma, float eps, uint8_t *q_packed,
                                          float *scale, float *sumsq_opt, float *ressq_opt,
                                          void *h_opt, void *stream)
{
    int rc = check_rows(x_f16, M, d, ldx, q_packed, scale);
    if (rc != QUOTA_OK) return rc;
    if (!gamma) return QUOTA_ERR_NULL;
    if (!(eps >= 0.0f)) return QUOTA_ERR_INVALID_ARG;
    if (M == 0) return QUOTA_OK;
    return rmsnorm_quantize(x_f16, M, d, ldx, gamma, eps, RowOutPacked{(uint32_t *)q_packed}, scale, sumsq_opt,
                            ressq_opt, h_opt, (hipStream_t)stream);
}

int quota_internal_rmsnorm_quantize_a6(const void *x_f16, int M, int d, const float *gamma, float eps, uint8_t *qa6,
                                       float *scale, float *sumsq_opt, float *ressq_opt, hipStream_t st, const quota_kept_copies *copies)
{
    int rc = check_rows(x_f16, M, d, d, qa6, scale);
    if (rc != QUOTA_OK) return rc;
    if (M == 0) return QUOTA_OK;
    if (copies) {                            // (quota_score_quantizes_beside: rows of at most 8192 columns, less than quota_a6_starts of them)
        if (quota_a6_starts(M) || d > 8192) return QUOTA_ERR_SHAPE;
        // (with the kept rows' codes and scales of K and V and their positions, read and written, and their numbers)
        const double kv = copies->dkv * (1 + 1.0 / 16);
        ProfScope prof(QUOTA_K_RMSNORM_QUANTIZE_ACT, 0, 2.5 * M * d + 4.0 * M + 4.0 * d + copies->rows * (2 * kv + 12), st);
        auto kernel = d <= 2048   ? rmsnorm_quantize_act_kernel<false, 256, 2, RowOutA6, quota_kept_copies>
                      : d <= 4096 ? rmsnorm_quantize_act_kernel<false, 512, 1, RowOutA6, quota_kept_copies>
                                  : rmsnorm_quantize_act_kernel<false, 512, 2, RowOutA6, quota_kept_copies>;
        kernel<<<dim3(M + copies->rows), dim3(d <= 2048 ? 256 : 512), 0, st>>>((const f16 *)x_f16, M, d, d, gamma, eps, RowOutA6{(uint32_t *)qa6}, scale, nullptr,
                                                                     nullptr, nullptr, *copies);
        QUOTA_RETURN_IF_LAUNCH_FAILED();
        return QUOTA_OK;
    }
    return with_a6_out(qa6, M, [&](auto out) { return rmsnorm_quantize(x_f16, M, d, d, gamma, eps, out, scale, sumsq_opt, ressq_opt, nullptr, st); });
}

template <typename OUT>
static int silu_mul_quantize(const void *gu_f16, int M, int F, OUT q, float *scale, void *z_opt,
                             const void *z_inject_opt, hipStream_t st)
{
    ProfScope prof(QUOTA_K_SILU_MUL_QUANTIZE_ACT, 0, 4.5 * M * F + 4.0 * M, st);
    with_row_shape<OUT>(M, F, [&](auto group, auto nch, dim3 grid) {
        constexpr bool can_be_early = group() >= 256 && nch() < 16;
        auto kernel = silu_mul_quantize_act_kernel<group(), nch(), can_be_early, OUT>;
        if constexpr (OUT::MANY && nch() > 2) {              // (two chunks: such a launch is the waves')
            if (M >= ROW_WAVE_MIN_ROWS) kernel = silu_mul_quantize_act_kernel<group(), nch(), false, OUT>;
        }
        kernel<<<grid, dim3(row_threads(group())), 0, st>>>((const f16 *)gu_f16, M, F, q, scale, (f16 *)z_opt, (const f16 *)z_inject_opt);
    });
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

extern "C" int quota_silu_mul_quantize_act(const void *gu_f16, int M, int F, uint8_t *q_packed,
                                           float *scale, void *z_opt, const void *z_inject_opt,
                                           void *stream)
{
    int rc = check_rows(gu_f16, M, F, F, q_packed, scale);
    if (rc != QUOTA_OK) return rc;
    if (M == 0) return QUOTA_OK;
    return silu_mul_quantize(gu_f16, M, F, RowOutPacked{(uint32_t *)q_packed}, scale, z_opt, z_inject_opt,
                             (hipStream_t)stream);
}

int quota_internal_silu_mul_quantize_a6(const void *gu_f16, int M, int F, uint8_t *qa6, float *scale,
                                        void *z_opt, const void *z_inject_opt, hipStream_t st)
{
    int rc = check_rows(gu_f16, M, F, F, qa6, scale);
    if (rc != QUOTA_OK) return rc;
    if (M == 0) return QUOTA_OK;
    return with_a6_out(qa6, M, [&](auto out) { return silu_mul_quantize(gu_f16, M, F, out, scale, z_opt, z_inject_opt, st); });
}

template <typename OUT>
static int quantize_rows(const void *x_f16, int M, int d, OUT q, float *scale, hipStream_t st)
{
    ProfScope prof(QUOTA_K_QUANTIZE_ACT, 0, 2.5 * M * d + 4.0 * M, st);
    with_row_shape<OUT>(M, d, [&](auto group, auto nch, dim3 grid) {
        quantize_act_kernel<false, group(), nch(), OUT><<<grid, dim3(row_threads(group())), 0, st>>>((const f16 *)x_f16, M, d, d, M, 0, q,
                                                                                            scale, nullptr, nullptr);
    });
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

// Per-token quantizer of a dense fp16 [M][d] into the A6 format.
int quota_internal_quantize_a6(const void *x_f16, int M, int d, uint8_t *qa6, float *scale, hipStream_t st)
{
    int rc = check_rows(x_f16, M, d, d, qa6, scale);
    if (rc != QUOTA_OK || M == 0) return rc;
    return with_a6_out(qa6, M, [&](auto out) { return quantize_rows(x_f16, M, d, out, scale, st); });
}

// The two quantizers of at most 32 rows into the few-row GEMM's fragments.
int quota_internal_rmsnorm_quantize_frag(const void *x_f16, int M, int d, const float *gamma, float eps, uint8_t *qf,
                                         float *scale, hipStream_t st)
{
    int rc = check_rows(x_f16, M, d, d, qf, scale);
    if (rc != QUOTA_OK || M == 0) return rc;
    return rmsnorm_quantize(x_f16, M, d, d, gamma, eps, RowOutFrag{(uint32_t *)qf}, scale, nullptr, nullptr, nullptr, st);
}
int quota_internal_quantize_frag(const void *x_f16, int M, int d, uint8_t *qf, float *scale, hipStream_t st)
{
    int rc = check_rows(x_f16, M, d, d, qf, scale);
    if (rc != QUOTA_OK || M == 0) return rc;
    return quantize_rows(x_f16, M, d, RowOutFrag{(uint32_t *)qf}, scale, st);
}

// Eq. 6 vector metrics only (no codes stored): sumsq/ressq [B][Nv] of the
// visual rows v[b][i] = v + b*stride_b + i*ldv.
int quota_internal_vector_metrics(const void *v_f16, int B, int Nv, int d, int ldv, long stride_b,
                                  float *sumsq, float *ressq, hipStream_t st)
{
    if (!v_f16 || !sumsq || !ressq) return QUOTA_ERR_NULL;
    if (B <= 0 || Nv < 0 || d <= 0) return QUOTA_ERR_INVALID_ARG;
    if (d % 8 != 0 || d > ROW_MAXCOLS || ldv < d || ldv % 8 != 0 || stride_b % 8 != 0)
        return QUOTA_ERR_SHAPE;
    if (Nv == 0) return QUOTA_OK;
    ProfScope prof(QUOTA_K_QUANTIZE_ACT, 0, 2.0 * B * Nv * d + 8.0 * B * Nv, st);
    with_row_shape<RowOutPacked>(B * Nv, d, [&](auto group, auto nch, dim3 grid) {
        quantize_act_kernel<true, group(), nch(), RowOutPacked><<<grid, dim3(row_threads(group())), 0, st>>>(
            (const f16 *)v_f16, B * Nv, d, ldv, Nv, stride_b, RowOutPacked{nullptr}, nullptr, sumsq, ressq);
    });
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}
