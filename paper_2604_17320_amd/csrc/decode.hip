// Decode-side kernels: one new token per sequence attends over the layer's pruned
// 4-bit KV cache (the cache that prefill wrote for retained tokens only), reading the
// codes and group scales straight from HBM and dequantizing them in registers.
// Bandwidth-bound by construction: a step moves H*dh + H*dh/16 bytes per cached token
// and sequence (K and V codes plus fp16 scales), a quarter of an fp16 cache.
#include <type_traits>
#include "common.h"
#include "internal.h"
#include "gemm_common.h"
#include "ropequant.h"
#include "ldsgrant.h"

namespace {

constexpr int DEC_LMAX = QUOTA_MAX_DECODE_ROWS;      // cached rows per sequence the decode calls accept

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// Dequantizes codes e and e+4 (e = 0..3) of a packed dword to x_hat = fp16(code * s) as a half
// pair.  wx = w ^ 0x88888888 turns each two's-complement nibble c into c + 8 in [0, 15];
// 0x6400 | (c + 8) is the fp16 number 1024 + c + 8, so subtracting 1032 leaves the code exactly,
// and the fp16 multiply rounds code * s once, to nearest -- the value the quantizer defines.
__device__ __forceinline__ h2 dequant_pair(uint32_t wx, int e, h2 s2)
{
    const uint32_t bits = ((wx >> (4 * e)) & 0x000F000Fu) | 0x64006400u;
    h2 c = __builtin_bit_cast(h2, bits);
    c = c - h2{(_Float16)1032.0f, (_Float16)1032.0f};
    return c * s2;
}

// The new token of a decode step, as the QKV projection left it (null qkv: the cache is read as it is).
struct DecodeNew {
    const f16 *qkv;             // [B][d + 2 dkv]
    const int32_t *pos;
    const float *cosT, *sinT;
    int n_pos;
    f16 *q_rot;                 // optional: also keep the rotated queries
};

// One workgroup per (sequence, K/V head, range of cached rows, RC query heads that share the K/V head),
// XCD-aware order; RC is 1 when every query head has its own K/V head, else 2.  The workgroups of a K/V
// head are neighbours on one XCD, so its rows come from HBM once and from that XCD's L2 afterwards.  The
// cached rows are walked in tiles of DEC_TILE tokens with a running softmax (maximum, sum, rescaled
// output), so the scores of one tile are all the LDS the walk needs, whatever the cache length.
//   new row: FUSED calls are handed the plain projection of the new token: wave 0 rotates q and k and
//            quantizes k and v while the first tile is on its way; the row is used from LDS, and one
//            workgroup per K/V head appends it to the cache (a launch less per layer, and the QKV GEMM
//            needs no epilogue);
//   loads:   the walk is latency-bound (a workgroup owns a few tens of KB), so every K and V load of a
//            tile is issued before the first use -- UN passes of 512 lanes x 16 bytes each -- and the next
//            tile's as soon as the registers of this one's are free;
//   scores:  DH/32 lanes per token, each holds 16 contiguous bytes of the token's K codes (32
//            channels) -- a wave reads whole 64- or 32-byte row segments -- dequantizes them as
//            packed fp16 pairs and dots them with the query; the lanes of a token add up by shuffles;
//   output:  the same lanes own 32 channels of V each and accumulate p * v_hat over their share of
//            the tokens; the token lanes are summed through LDS in a fixed order at the end.
// step_dev (optional): the cache length is len + *step_dev + 1 (a HIP-graph-captured decode loop keeps
// its step count on the device).
// SPLIT: n_split workgroups share a K/V head's rows, `tiles` tiles each; they leave unnormalized outputs,
// maxima and sums in `part` for decode_combine_kernel.
constexpr int DEC_TILE = 512;
constexpr int DEC_THREADS = 512;     // 8 waves: with two workgroups on a CU every SIMD has four waves to interleave
constexpr int DEC_RED_ROW = DEC_THREADS + 1;

template <int DH, int RC, bool FUSED, bool SPLIT>
__global__ __launch_bounds__(DEC_THREADS, RC == 1 ? 4 : 2) void decode_attention_kernel(
    const f16 *__restrict__ q, int d, int dkv, int rep, uint32_t *__restrict__ kc, f16 *__restrict__ ks,
    uint32_t *__restrict__ vc, f16 *__restrict__ vs, int capacity, int len,
    const int32_t *__restrict__ step_dev, int max_steps, f16 *__restrict__ o, int n_kv_heads, DecodeNew nw,
    int n_split, int tiles, float *__restrict__ part)
{
    constexpr int PPT = DH / 32;            // 16-byte pieces (lanes) per token and head
    constexpr int TP = DEC_THREADS / PPT;   // tokens per pass of the workgroup
    constexpr int UN = DEC_TILE / TP;       // passes per tile
    constexpr int WPT = DH / 8;             // packed dwords per token and head
    constexpr int GPT = DH / 64;            // scale groups per token and head
    constexpr int NW = DEC_THREADS / 64;    // waves
    extern __shared__ float red[];          // [32 channels][512 token lanes], padded
    __shared__ h2 qp[RC][DH / 2];           // q as pairs: qp[r][4 i + e] = (q[8 i + e], q[8 i + e + 4])
    __shared__ float sc[RC][DEC_TILE];
    __shared__ float wred[2][RC][NW];
    __shared__ __align__(16) uint32_t new_codes[2][WPT];
    __shared__ f16 new_scales[2][GPT];
    // (sequence, head) pairs are dealt to the 8 XCDs in contiguous ranges: the heads of a sequence
    // share the 128-byte lines of its cache rows (two heads' codes, all heads' scales), and each
    // XCD has its own L2
    const int n_pass = (rep + RC - 1) / RC;            // workgroups per K/V head: RC query heads each
    const int work = xcd_remap(blockIdx.x, gridDim.x);
    const int r0 = (work % n_pass) * RC;
    const int sp = SPLIT ? work / n_pass % n_split : 0;
    const int bh = work / (SPLIT ? n_pass * n_split : n_pass), h = bh % n_kv_heads, b = bh / n_kv_heads;
    const int tid = threadIdx.x, wave = tid >> 6;
    const int piece = tid % PPT, tl = tid / PPT;
    const int wave_t0 = (tid & ~63) / PPT;  // first token of this wave within a pass
    const int n32 = dkv >> 3, ng = dkv >> 6;
    int L = len;
    if (step_dev) L += min(max(*step_dev, 0), max_steps - 1) + 1;      // the row this step appends included
    const int stored = FUSED ? L - 1 : L;   // rows read from the cache
    const int t_begin = SPLIT ? sp * tiles * DEC_TILE : 0, t_end = SPLIT ? min(t_begin + tiles * DEC_TILE, L) : L;
    const float scale = 1.0f / sqrtf((float)DH);
    const size_t row0 = (size_t)b * capacity;
    const int nr = min(RC, rep - r0);

    uint4 kq[UN], vq[UN];
    f16 ksc[UN], vsc[UN];
    auto load_k = [&](int t0) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int t = t0 + u * TP + tl;
            const size_t row = row0 + (t < stored ? t : 0);
            kq[u] = *reinterpret_cast<const uint4 *>(kc + row * n32 + h * WPT + 4 * piece);
            ksc[u] = ks[row * ng + h * GPT + (piece >> 1)];
        }
    };
    auto load_v = [&](int t0) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int t = t0 + u * TP + tl;
            const size_t row = row0 + (t < stored ? t : 0);
            vq[u] = *reinterpret_cast<const uint4 *>(vc + row * n32 + h * WPT + 4 * piece);
            vsc[u] = vs[row * ng + h * GPT + (piece >> 1)];
        }
    };
    Pack16 x, xp, xo;
    float cs[8], sn[8];
    constexpr int CPH = DH / 8, HALF = CPH / 2;
    const int item = tid / CPH, cc = tid % CPH;         // wave 0: head vectors k, v, q[0], q[1]
    if (FUSED) {
        // its loads go first: they head the longest chain
        if (tid < (2 + RC) * CPH) {
            const int hq = h * rep + min(r0 + max(item - 2, 0), rep - 1);
            const int first = item == 0 ? d + h * DH : item == 1 ? d + dkv + h * DH : hq * DH;
            x.u = *reinterpret_cast<const uint4 *>(nw.qkv + (size_t)b * (d + 2 * dkv) + first + 8 * cc);
            const int pr = min(max(nw.pos[b], 0), nw.n_pos - 1);     // never index outside the tables
            const float *cp = nw.cosT + (size_t)pr * (DH / 2) + 8 * (cc % HALF);
            const float *ssp = nw.sinT + (size_t)pr * (DH / 2) + 8 * (cc % HALF);
            *reinterpret_cast<float4 *>(cs) = *reinterpret_cast<const float4 *>(cp);
            *reinterpret_cast<float4 *>(cs + 4) = *reinterpret_cast<const float4 *>(cp + 4);
            *reinterpret_cast<float4 *>(sn) = *reinterpret_cast<const float4 *>(ssp);
            *reinterpret_cast<float4 *>(sn + 4) = *reinterpret_cast<const float4 *>(ssp + 4);
        }
    }
    load_k(t_begin);
    load_v(t_begin);
    if (FUSED) {
        if (tid < (2 + RC) * CPH) {
#pragma unroll
            for (int i = 0; i < 4; ++i) xp.w[i] = __shfl_xor(x.w[i], HALF, 64);     // rotate-half partner chunk
            if (item == 1) xo = x;
            else rope8(x, xp, cs, sn, cc >= HALF, xo);
            if (item < 2) {
                float f[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = (float)xo.h[e];
                f16 s8;
                const uint32_t word = kv_quant8(f, &s8, nullptr);
                new_codes[item][cc] = word;
                if ((cc & 7) == 0) new_scales[item][cc >> 3] = s8;
                if (r0 == 0 && L > t_begin && L <= t_end) {
                    const size_t row = row0 + L - 1;
                    (item == 0 ? kc : vc)[row * n32 + h * WPT + cc] = word;
                    if ((cc & 7) == 0) (item == 0 ? ks : vs)[row * ng + h * GPT + (cc >> 3)] = s8;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) qp[item - 2][4 * cc + e] = h2{xo.h[e], xo.h[e + 4]};
                if (nw.q_rot && sp == 0 && item - 2 < nr)
                    *reinterpret_cast<uint4 *>(nw.q_rot + (size_t)b * d + (h * rep + r0 + item - 2) * DH + 8 * cc) = xo.u;
            }
        }
    } else if (tid < RC * (DH / 2)) {
        const int r = tid / (DH / 2), i = tid % (DH / 2);
        const int hq = min(h * rep + r0 + r, h * rep + rep - 1);
        const f16 *qh = q + (size_t)b * d + hq * DH + 8 * (i >> 2) + (i & 3);
        qp[r][i] = h2{qh[0], qh[4]};
    }
    __syncthreads();
    h2 qr[RC][16];                      // this lane's 32 channels of each query, as pairs
#pragma unroll
    for (int r = 0; r < RC; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) qr[r][i] = qp[r][16 * piece + i];
    float m_run[RC], l_run[RC], acc[RC][32];
#pragma unroll
    for (int r = 0; r < RC; ++r) {
        m_run[r] = -INFINITY;
        l_run[r] = 0.0f;
#pragma unroll
        for (int e = 0; e < 32; ++e) acc[r][e] = 0.0f;
    }
    for (int t0 = t_begin; t0 < t_end; t0 += DEC_TILE) {
        const int tn = min(DEC_TILE, t_end - t0);
        if (FUSED && t0 + tn == L) {    // the new row is in this tile
#pragma unroll
            for (int u = 0; u < UN; ++u)
                if (t0 + u * TP + tl == L - 1) {
                    kq[u] = *reinterpret_cast<const uint4 *>(&new_codes[0][4 * piece]);
                    vq[u] = *reinterpret_cast<const uint4 *>(&new_codes[1][4 * piece]);
                    ksc[u] = new_scales[0][piece >> 1];
                    vsc[u] = new_scales[1][piece >> 1];
                }
        }
        // ---- scores of the tile
        float mx[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) mx[r] = -INFINITY;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (u * TP + wave_t0 >= tn) continue;       // the whole wave is past the end
            const int t = u * TP + tl;
            const bool ok = t < tn;
            const h2 s2 = h2{ksc[u], ksc[u]};
            const uint32_t ww[4] = {kq[u].x ^ 0x88888888u, kq[u].y ^ 0x88888888u, kq[u].z ^ 0x88888888u,
                                    kq[u].w ^ 0x88888888u};
            float dot[RC][4];           // four independent chains: the dot instruction accumulates in place
#pragma unroll
            for (int r = 0; r < RC; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) dot[r][i] = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) {       // channels (8 id + e, 8 id + e + 4), id = 4 piece + i
                    const h2 kh = dequant_pair(ww[i], e, s2);
#pragma unroll
                    for (int r = 0; r < RC; ++r)
                        dot[r][i] = __builtin_amdgcn_fdot2(qr[r][4 * i + e], kh, dot[r][i], false);
                }
#pragma unroll
            for (int r = 0; r < RC; ++r) {
                float v = (dot[r][0] + dot[r][1]) + (dot[r][2] + dot[r][3]);
                v += __shfl_xor(v, 1, 64);
                if (PPT == 4) v += __shfl_xor(v, 2, 64);
                v *= scale;
                if (ok && piece == 0) sc[r][t] = v;
                if (ok) mx[r] = fmaxf(mx[r], v);
            }
        }
        const bool more = t0 + DEC_TILE < t_end;
        if (more) load_k(t0 + DEC_TILE);
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            mx[r] = wave_max(mx[r]);
            if ((tid & 63) == 0) wred[0][r][wave] = mx[r];
        }
        __syncthreads();                // scores and wave maxima visible
        float alpha[RC], m_new[RC], sum[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            float tm = wred[0][r][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) tm = fmaxf(tm, wred[0][r][w]);
            m_new[r] = fmaxf(m_run[r], tm);
            alpha[r] = __expf(m_run[r] - m_new[r]);      // 0 on the first tile
            m_run[r] = m_new[r];
            sum[r] = 0.0f;
            for (int t = tid; t < tn; t += DEC_THREADS) {
                const float p = __expf(sc[r][t] - m_new[r]);
                sc[r][t] = p;
                sum[r] += p;
            }
            sum[r] = wave_sum(sum[r]);
            if ((tid & 63) == 0) wred[1][r][wave] = sum[r];
        }
        __syncthreads();                // probabilities and wave sums visible
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            float ts = wred[1][r][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) ts += wred[1][r][w];
            l_run[r] = l_run[r] * alpha[r] + ts;
#pragma unroll
            for (int e = 0; e < 32; ++e) acc[r][e] *= alpha[r];
        }
        // ---- p * v_hat of the tile
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (u * TP + wave_t0 >= tn) continue;
            const int t = u * TP + tl;
            const bool ok = t < tn;
            const h2 s2 = h2{vsc[u], vsc[u]};
            const uint32_t ww[4] = {vq[u].x ^ 0x88888888u, vq[u].y ^ 0x88888888u, vq[u].z ^ 0x88888888u,
                                    vq[u].w ^ 0x88888888u};
            float pv[RC];
#pragma unroll
            for (int r = 0; r < RC; ++r) pv[r] = ok ? sc[r][t] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const h2 vh = dequant_pair(ww[i], e, s2);
#pragma unroll
                    for (int r = 0; r < RC; ++r) {
                        acc[r][8 * i + e] = fmaf(pv[r], (float)vh[0], acc[r][8 * i + e]);
                        acc[r][8 * i + e + 4] = fmaf(pv[r], (float)vh[1], acc[r][8 * i + e + 4]);
                    }
                }
        }
        if (more) {
            load_v(t0 + DEC_TILE);
            __syncthreads();            // the tile's scores have been consumed
        }
    }
    // ---- the token lanes meet in LDS, summed in lane order (red is laid out [channel][token lane] so that
    // the lanes of a wave write consecutive words; the loop over r is unrolled to keep acc in registers)
#pragma unroll
    for (int r = 0; r < RC; ++r) {
        if (r >= nr) break;
        if (r) __syncthreads();
#pragma unroll
        for (int e = 0; e < 32; ++e) red[e * DEC_RED_ROW + tid] = acc[r][e];
        __syncthreads();
        if (tid < DH) {
            float out = 0.0f;
            const float *rp = red + (tid & 31) * DEC_RED_ROW + (tid >> 5);
#pragma unroll 32
            for (int i = 0; i < TP; ++i) out += rp[i * PPT];
            const int hq = h * rep + r0 + r;
            if (SPLIT) {
                float *p = part + ((size_t)(b * n_kv_heads * rep + hq) * n_split + sp) * (DH + 2);
                p[tid] = out;
                if (tid == 0) { p[DH] = m_run[r]; p[DH + 1] = l_run[r]; }
            } else {
                o[(size_t)b * d + hq * DH + tid] = (f16)(out / l_run[r]);
            }
        }
    }
}

// One workgroup per (sequence, query head): the splits' outputs under a common maximum.
template <int DH>
__global__ __launch_bounds__(DH) void decode_combine_kernel(const float *__restrict__ part, int n_split, f16 *__restrict__ o)
{
    const float *p = part + (size_t)blockIdx.x * n_split * (DH + 2);
    float m = -INFINITY, l = 0.0f, out = 0.0f;
    for (int s = 0; s < n_split; ++s) m = fmaxf(m, p[s * (DH + 2) + DH]);
    for (int s = 0; s < n_split; ++s) {
        const float a = __expf(p[s * (DH + 2) + DH] - m);       // 0 for a split without rows
        l = __builtin_fmaf(a, p[s * (DH + 2) + DH + 1], l);
        out = __builtin_fmaf(a, p[s * (DH + 2) + threadIdx.x], out);
    }
    o[(size_t)blockIdx.x * DH + threadIdx.x] = (f16)(out / l);
}

constexpr int DEC_SPLIT_ROWS = 1024, DEC_SPLIT_GRID = 256;

template <int DH, bool FUSED>
int launch_decode(const f16 *q, int Hq, const quota_kv_cache *c, int len, f16 *o, const DecodeNew &nw, float *part,
                  hipStream_t st)
{
    const int d = Hq * DH, dkv = c->H * DH, rep = Hq / c->H, rc = rep == 1 ? 1 : 2;
    const bool stepped = c->step_dev != nullptr;
    const int longest = stepped ? c->len + c->max_steps : len;
    const double rows = (double)c->B * longest;
    ProfScope prof(QUOTA_K_ATTENTION_DECODE, 4.0 * rows * d, rows * (dkv + dkv / 16.0) + 4.0 * c->B * d, st);
    const int heads = c->H * c->B * ((rep + rc - 1) / rc), n_tiles = (longest + DEC_TILE - 1) / DEC_TILE;
    int n_split = 1, tiles = n_tiles;
    if (part && longest > DEC_SPLIT_ROWS && heads < DEC_SPLIT_GRID) {
        tiles = max(1, n_tiles * heads / (2 * DEC_SPLIT_GRID));
        n_split = (n_tiles + tiles - 1) / tiles;
    }
    auto run = [&](auto kernel_tag) {
        constexpr auto kernel = decltype(kernel_tag)::value;
        constexpr size_t lds = 32 * DEC_RED_ROW * sizeof(float);
        if (!grant_lds<kernel>()) return QUOTA_ERR_HIP;
        kernel<<<dim3(heads * n_split), dim3(DEC_THREADS), lds, st>>>(
            q, d, dkv, rep, (uint32_t *)c->k_codes, (f16 *)c->k_scales, (uint32_t *)c->v_codes, (f16 *)c->v_scales,
            c->capacity, stepped ? c->len : len, c->step_dev, c->max_steps, o, c->H, nw, n_split, tiles, part);
        QUOTA_RETURN_IF_LAUNCH_FAILED();
        return QUOTA_OK;
    };
#define KERNEL(RC, SPLIT) std::integral_constant<decltype(&decode_attention_kernel<DH, RC, FUSED, SPLIT>), \
                                                 &decode_attention_kernel<DH, RC, FUSED, SPLIT>>()
    if constexpr (FUSED) {
        if (n_split > 1) {
            const int rcode = rep == 1 ? run(KERNEL(1, true)) : run(KERNEL(2, true));
            if (rcode != QUOTA_OK) return rcode;
            decode_combine_kernel<DH><<<dim3(c->B * Hq), dim3(DH), 0, st>>>(part, n_split, o);
            QUOTA_RETURN_IF_LAUNCH_FAILED();
            return QUOTA_OK;
        }
    }
    return rep == 1 ? run(KERNEL(1, false)) : run(KERNEL(2, false));
#undef KERNEL
}

__global__ void advance_step_kernel(int32_t *step) { *step += 1; }

}  // namespace

int quota_internal_advance_step(int32_t *step_dev, hipStream_t st)
{
    advance_step_kernel<<<1, 1, 0, st>>>(step_dev);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

extern "C" int quota_advance_step(int32_t *step_dev, void *stream)
{
    if (!step_dev) return QUOTA_ERR_NULL;
    return quota_internal_advance_step(step_dev, (hipStream_t)stream);
}

size_t quota_internal_decode_part_bytes(int B, int H, int Hkv, int dh)
{
    const int rep = H / Hkv, heads = Hkv * B * (rep == 1 ? 1 : (rep + 1) / 2);
    return heads < DEC_SPLIT_GRID ? (size_t)B * H * (DEC_LMAX / DEC_TILE) * (dh + 2) * sizeof(float) : 0;
}

int quota_internal_attention_decode_new(const void *qkv_f16, const int32_t *pos, const float *cosT, const float *sinT,
                                        int n_pos, int Hq, const quota_kv_cache *cache, void *q_rot_opt, void *o_f16,
                                        void *part, hipStream_t st)
{
    const DecodeNew nw = {(const f16 *)qkv_f16, pos, cosT, sinT, n_pos, (f16 *)q_rot_opt};
    return cache->dh == 128
               ? launch_decode<128, true>(nullptr, Hq, cache, cache->len + 1, (f16 *)o_f16, nw, (float *)part, st)
               : launch_decode<64, true>(nullptr, Hq, cache, cache->len + 1, (f16 *)o_f16, nw, (float *)part, st);
}

extern "C" int quota_attention_decode_gqa(const void *q_f16, int Hq, const quota_kv_cache *cache,
                                          void *o_f16, void *stream)
{
    if (!q_f16 || !cache || !o_f16 || !cache->k_codes || !cache->k_scales || !cache->v_codes ||
        !cache->v_scales)
        return QUOTA_ERR_NULL;
    const bool stepped = cache->step_dev != nullptr;     // length = len + *step_dev + 1 (read on the device)
    if (cache->B <= 0 || cache->H <= 0 || Hq <= 0 || cache->len > cache->capacity ||
        (stepped ? cache->len < 0 || cache->max_steps <= 0 || cache->len + cache->max_steps > cache->capacity
                 : cache->len <= 0))
        return QUOTA_ERR_INVALID_ARG;
    const int longest = stepped ? cache->len + cache->max_steps : cache->len;
    if ((cache->dh != 64 && cache->dh != 128) || longest > DEC_LMAX || Hq % cache->H != 0)
        return QUOTA_ERR_SHAPE;
    const DecodeNew none = {};
    return cache->dh == 128
               ? launch_decode<128, false>((const f16 *)q_f16, Hq, cache, cache->len, (f16 *)o_f16, none, nullptr,
                                           (hipStream_t)stream)
               : launch_decode<64, false>((const f16 *)q_f16, Hq, cache, cache->len, (f16 *)o_f16, none, nullptr,
                                          (hipStream_t)stream);
}

extern "C" int quota_attention_decode(const void *q_f16, const quota_kv_cache *cache, void *o_f16,
                                      void *stream)
{
    if (!cache) return QUOTA_ERR_NULL;
    return quota_attention_decode_gqa(q_f16, cache->H, cache, o_f16, stream);
}
