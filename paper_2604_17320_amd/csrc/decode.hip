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

// Dequantizes a packed dword to x_hat = fp16(code * s): pair e holds codes e and e + 4.  A two's-complement nibble c
// under 0x6400 | . ^ 8 is the fp16 number 1024 + c + 8, a nibble one place up (0x6400 | . ^ 0x80) is 1024 +
// 16 (c + 8): one subtraction, or one multiply-add by 1/16, leaves the code exactly, and the fp16 multiply
// rounds code * s once, to nearest -- the value the quantizer defines.  13 instructions per 8 codes
// (the masks sit in registers, so that and + xor is one instruction).
struct Dequant {
    uint32_t m0 = 0x000F000Fu, m1 = 0x00F000F0u, x0 = 0x64086408u, x1 = 0x64806480u;
    __device__ __forceinline__ Dequant() { asm volatile("" : "+v"(m0), "+v"(m1), "+v"(x0), "+v"(x1)); }
    __device__ __forceinline__ void operator()(uint32_t w, h2 s2, h2 out[4]) const
    {
        const h2 sixteenth = h2{(_Float16)0.0625f, (_Float16)0.0625f};
        const uint32_t hi = w >> 8;
        const uint32_t b[4] = {(w & m0) ^ x0, (w & m1) ^ x1, (hi & m0) ^ x0, (hi & m1) ^ x1};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const h2 v = __builtin_bit_cast(h2, b[e]);
            out[e] = (e & 1 ? __builtin_elementwise_fma(v, sixteenth, h2{(_Float16)-72.0f, (_Float16)-72.0f})
                            : v - h2{(_Float16)1032.0f, (_Float16)1032.0f}) * s2;
        }
    }
};

// The value of another lane of the quad
template <int CTRL>
__device__ __forceinline__ float quad_swap(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
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
//   new row: FUSED calls are handed the plain projection of the new token: a workgroup's first
//            threads rotate q and k and quantize k and v while the first tile is on its way; the row is
//            used from LDS, and one workgroup per K/V head appends it to the cache (a launch less per
//            layer, and the QKV GEMM needs no epilogue);
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
// VS > 1: so many workgroups share the channels of V of a head, each with all scores: a lane's piece is 32 / VS channels, which makes
// the products with V and the sum over the token lanes, two fifths of the instructions, shorter and leaves every sum in its order (the
// same bits).  For launches that leave CUs idle.  Asked for beside K, or the next tile's K before the softmax, V and K make the step
// slower (1260 -> 1281 us, 1264).
// SPLIT: n_split workgroups share a K/V head's rows, split_tiles() tiles each; they leave unnormalized outputs,
// maxima and sums in `part` for decode_combine_kernel.
constexpr int DEC_TILE = 512;
constexpr int DEC_SPLIT_GRID = 256;
// Tiles per workgroup when rows of n_tiles tiles are walked by `heads` workgroups, or by more where they are split.
// Few heads over long caches: split so that every workgroup still has a CU to itself, if that saves two tiles of the walk or
// more (a tile takes 4.5 us, the combining launch 3: 3 sequences of 4003 rows, 4 K/V heads: 44 us unsplit, 25 in
// 384 workgroups of one tile, 19 in 192 of two).  The split is the order of the sums: it goes by the rows there are, on
// the device too, so that a step of a captured loop leaves the bits of the call with a host-side length.  (A first part that
// holds all the rows leaves the bits of the unsplit walk, the empty ones behind it count as nothing.)
__host__ __device__ inline int split_tiles(int n_tiles, int heads)
{
    const int t = (n_tiles * heads + DEC_SPLIT_GRID - 1) / DEC_SPLIT_GRID;
    return n_tiles - t >= 2 ? t : n_tiles;
}
constexpr int DEC_THREADS = 512;     // 8 waves: with two workgroups on a CU every SIMD has four waves to interleave
// A head's sums per token lane on their way to one thread per channel: a row of token lanes per channel, read 16 bytes
// at a time (4 bytes at a time 128 reads were 0.3 us longer), its start moved on by piece so that a wave's 64 writes
// fall on 64 banks.
constexpr int dec_red_row(int dh) { return DEC_THREADS / (dh / 32) + 4; }
constexpr int dec_red_floats(int dh, int hp, int vs) { return hp * dh / vs * dec_red_row(dh) + 64; }

template <int DH, int RC, int HP, bool MULTI, bool FUSED, bool SPLIT, int VS>
__global__ __launch_bounds__(HP * DEC_THREADS, RC == 1 && !SPLIT ? 4 : 2) void decode_attention_kernel(
    const int32_t *__restrict__ step_dev, const int32_t *__restrict__ pos, int wgs, int n_kv_heads, int rep_arg, int n_split, int d, int dkv,
    const f16 *__restrict__ q, uint32_t *__restrict__ kc, f16 *__restrict__ ks, uint32_t *__restrict__ vc, f16 *__restrict__ vs, int capacity, int len,
    int max_steps, int heads, f16 *__restrict__ o, DecodeNew nw, float *__restrict__ part)
{
    // The step count (without one: any number there is) and the new token's position are asked for together, before anything else needs them: by scalar loads,
    // from address space 4, since nothing writes them while the kernel runs.
    typedef const __attribute__((address_space(4))) int32_t *scalar_i32;
    const int rep = RC == 1 ? 1 : rep_arg;
    int step = 0;
    if (FUSED || step_dev) step = *(scalar_i32)(uint64_t)(FUSED && !step_dev ? pos : step_dev);
    constexpr int PPT = DH / 32;            // 16-byte pieces (lanes) per token and head
    constexpr int TP = DEC_THREADS / PPT;   // tokens per pass of the workgroup
    constexpr int UN = DEC_TILE / TP;       // passes per tile
    constexpr int WPT = DH / 8;             // packed dwords per token and head
    constexpr int GPT = DH / 64;            // scale groups per token and head
    constexpr int NW = HP * DEC_THREADS / 64;       // waves
    static_assert(HP == 1 || (RC == 1 && !SPLIT), "");
    static_assert(VS == 1 || ((VS == 2 || VS == 4) && HP == 1 && !SPLIT && FUSED), "");
    constexpr int VC = 32 / VS, VD = 4 / VS;    // channels and dwords of V per lane
    extern __shared__ __align__(16) float red[];    // dec_red_floats
    constexpr int RROW = dec_red_row(DH);
    __shared__ h2 qp[HP * RC][DH / 2];      // q as pairs: qp[r][4 i + e] = (q[8 i + e], q[8 i + e + 4])
    __shared__ float sc[HP * RC][DEC_TILE];
    __shared__ float lsum[HP];
    __shared__ float wmax[HP * RC][NW], wsum[HP * RC][NW / HP];
    __shared__ __align__(16) uint32_t new_codes[2][HP * WPT];
    __shared__ __align__(4) f16 new_scales[2][HP * GPT];
    // (sequence, head) pairs are dealt to the 8 XCDs in contiguous ranges: the heads of a sequence
    // share the 128-byte lines of its cache rows (two heads' codes, all heads' scales), and each
    // XCD has its own L2
    const unsigned n_pass = RC == 1 ? 1u : (unsigned)(rep + RC - 1) / RC;            // workgroups per K/V head: RC query heads each
    const unsigned work = xcd_remap(blockIdx.x, wgs), passes = work / n_pass;
    const int r0 = (int)(work - passes * n_pass) * RC;
    const unsigned parts = SPLIT ? n_split : VS, own = passes / parts;
    const int sp = SPLIT ? (int)(passes - own * parts) : 0;
    const int vsp = VS > 1 ? (int)(passes - own * parts) : 0;         // this workgroup's dwords of every piece of V
    const unsigned bh = own * HP;
    const int b = (int)(bh / (unsigned)n_kv_heads), h = (int)(bh - b * (unsigned)n_kv_heads);        // (first) K/V head
    const int new_pos = FUSED ? ((scalar_i32)(uint64_t)pos)[b] : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int piece = tid % PPT, hs = tid / PPT % HP, tl = tid / (PPT * HP);
    constexpr int TPW = 64 / (PPT * HP);    // tokens per pass of a wave
    const int wave_t0 = wave * TPW;         // first token of this wave within a pass
    const int n32 = dkv >> 3, ng = dkv >> 6;
    int L = len;
    if (step_dev) L += min(max(step, 0), max_steps - 1) + 1;      // the row this step appends included
    const int stored = FUSED ? L - 1 : L;   // rows read from the cache
    const int share = SPLIT ? split_tiles((L + DEC_TILE - 1) / DEC_TILE, heads) * DEC_TILE : L;
    const int t_begin = SPLIT ? sp * share : 0, t_end = SPLIT ? min(t_begin + share, L) : L;
    const float scale = 1.0f / sqrtf((float)DH);
    const size_t row0 = (size_t)b * capacity;
    const int nr = min(RC, rep - r0);
    const Dequant dequant;

    // Loads are buffer loads that fetch nothing past the last row, so that every pass issues the same instructions
    // and waits count exactly.  The scales of a wave's tokens come 64 / HP tokens to a load (lane l: head l % HP, the
    // (l / HP)-th of the tokens of a tile) and are handed round the wave.
    const int rows = SPLIT ? min(stored, t_end) : stored;
    auto buffer = [&](const void *base, size_t row_bytes, int bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0,
                                                 rows > 0 ? (int)((rows - 1) * row_bytes + bytes) : 0, 0x00020000);
    };
    const auto kbuf = buffer(kc + row0 * n32 + h * WPT, 4 * n32, HP * WPT * 4);
    const auto vbuf = buffer(vc + row0 * n32 + h * WPT, 4 * n32, HP * WPT * 4);
    const auto ksbuf = buffer(ks + row0 * ng + h * GPT, 2 * ng, HP * GPT * 2);
    const auto vsbuf = buffer(vs + row0 * ng + h * GPT, 2 * ng, HP * GPT * 2);
    i32x4 slot[UN];                     // codes of a pass: K until its scores are taken, then V
    uint32_t vword[VS > 1 ? UN : 1][VD];        // VS > 1: V has registers of its own
    uint32_t ksw, vsw;
    const int scale_t = (lane / HP / TPW) * TP + wave_t0 + lane / HP % TPW;
    const int code_off = tl * (4 * n32) + 16 * (tid % (PPT * HP)), scale_off = scale_t * (2 * ng) + lane % HP * (2 * GPT);
    // (the opaque token number keeps the compiler from carrying every pass's offset in a register of its own)
    auto load_codes = [&](auto buf, int t) {
        asm volatile("" : "+s"(t));
        return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, code_off + t * (4 * n32), 0, 0));
    };
    auto load_vwords = [&](uint32_t (&v)[VD], int t) {
        asm volatile("" : "+s"(t));
        const int at = code_off + 4 * VD * vsp + t * (4 * n32);
        if constexpr (VD == 2) {
            const auto two = __builtin_amdgcn_raw_buffer_load_b64(vbuf, at, 0, 0);
            v[0] = two[0];
            v[1] = two[1];
        } else {
            v[0] = __builtin_amdgcn_raw_buffer_load_b32(vbuf, at, 0, 0);
        }
    };
    auto load_scales = [&](auto buf, int t) -> uint32_t {
        asm volatile("" : "+s"(t));
        if constexpr (GPT == 2) return __builtin_amdgcn_raw_buffer_load_b32(buf, scale_off + t * (2 * ng), 0, 0);
        else return __builtin_amdgcn_raw_buffer_load_b16(buf, scale_off + t * (2 * ng), 0, 0);
    };
    const uint32_t scale_sel = GPT == 2 && piece >= 2 ? 0x03020302u : 0x01000100u;
    const int scale_from = 4 * (HP * (lane / (PPT * HP)) + hs);
    auto scale_of = [&](uint32_t sw, int u) {       // of pass u's token, as a pair
        int from = scale_from;
        asm volatile("" : "+v"(from));              // (recomputed per pass, not kept for each)
        const uint32_t v = (uint32_t)__builtin_amdgcn_ds_bpermute(from + 4 * HP * TPW * u, (int)sw);
        return __builtin_bit_cast(h2, __builtin_amdgcn_perm(v, v, scale_sel));
    };
    Pack16 x, xp, xo;
    float cs[8], sn[8];
    constexpr int CPH = DH / 8, HALF = CPH / 2;
    const int item = tid / CPH % (2 + RC), cc = tid % CPH;          // head vectors k, v, q[0], q[1] ...
    const int ph = tid / CPH / (2 + RC);                            // ... of head h + ph
    const bool preparing = tid < HP * (2 + RC) * CPH;
    if (FUSED) {
        if (preparing) {
            const int hq = (h + ph) * rep + min(r0 + max(item - 2, 0), rep - 1);
            const int first = item == 0 ? d + (h + ph) * DH : item == 1 ? d + dkv + (h + ph) * DH : hq * DH;
            x.u = *reinterpret_cast<const uint4 *>(nw.qkv + (size_t)b * (d + 2 * dkv) + first + 8 * cc);
            const int pr = min(max(new_pos, 0), nw.n_pos - 1);       // never index outside the tables
            const float *cp = nw.cosT + (size_t)pr * (DH / 2) + 8 * (cc % HALF);
            const float *ssp = nw.sinT + (size_t)pr * (DH / 2) + 8 * (cc % HALF);
            *reinterpret_cast<float4 *>(cs) = *reinterpret_cast<const float4 *>(cp);
            *reinterpret_cast<float4 *>(cs + 4) = *reinterpret_cast<const float4 *>(cp + 4);
            *reinterpret_cast<float4 *>(sn) = *reinterpret_cast<const float4 *>(ssp);
            *reinterpret_cast<float4 *>(sn + 4) = *reinterpret_cast<const float4 *>(ssp + 4);
        }
        // (loads return in order: position, then angles, behind the tile's would wait for all of it; 16 sequences of 700 rows,
        // 32 heads: 17.9 -> 16.7 us)
        __builtin_amdgcn_sched_barrier(0);
    }
    ksw = load_scales(ksbuf, t_begin);
#pragma unroll
    for (int u = 0; u < UN; ++u) slot[u] = load_codes(kbuf, t_begin + u * TP);
    if (FUSED) {
        if (preparing) {
#pragma unroll
            for (int i = 0; i < 4; ++i) xp.w[i] = __shfl_xor(x.w[i], HALF, 64);     // rotate-half partner chunk
            if (item == 1) xo = x;
            else rope8(x, xp, cs, sn, cc >= HALF, xo);
            if (item < 2) {
                f16 s8;
                const uint32_t word = kv_quant8(xo, &s8, nullptr);
                new_codes[item][ph * WPT + cc] = word;
                if ((cc & 7) == 0) new_scales[item][ph * GPT + (cc >> 3)] = s8;
                if (r0 == 0 && vsp == 0 && L > t_begin && L <= t_end) {
                    const size_t row = row0 + L - 1;
                    (item == 0 ? kc : vc)[row * n32 + (h + ph) * WPT + cc] = word;
                    if ((cc & 7) == 0) (item == 0 ? ks : vs)[row * ng + (h + ph) * GPT + (cc >> 3)] = s8;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) qp[ph * RC + item - 2][4 * cc + e] = h2{xo.h[e], xo.h[e + 4]};
                if (nw.q_rot && sp == 0 && vsp == 0 && item - 2 < nr)
                    *reinterpret_cast<uint4 *>(nw.q_rot + (size_t)b * d + ((h + ph) * rep + r0 + item - 2) * DH + 8 * cc) = xo.u;
            }
        }
    } else if (tid < HP * RC * (DH / 2)) {
        const int r = tid / (DH / 2), i = tid % (DH / 2);
        const int hq = (h + r / RC) * rep + min(r0 + r % RC, rep - 1);
        const f16 *qh = q + (size_t)b * d + hq * DH + 8 * (i >> 2) + (i & 3);
        qp[r][i] = h2{qh[0], qh[4]};
    }
    __syncthreads();
    h2 qr[RC][16];                      // this lane's 32 channels of each query, as pairs
#pragma unroll
    for (int r = 0; r < RC; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) qr[r][i] = qp[hs * RC + r][16 * piece + i];
    float m_run[HP * RC], l_run[RC], acc[RC][VC];
#pragma unroll
    for (int r = 0; r < HP * RC; ++r) m_run[r] = -INFINITY;
#pragma unroll
    for (int r = 0; r < RC; ++r) {
        l_run[r] = 0.0f;
#pragma unroll
        for (int e = 0; e < VC; ++e) acc[r][e] = 0.0f;
    }
    for (int t0 = t_begin; t0 < t_end; t0 += DEC_TILE) {
        const int tn = min(DEC_TILE, t_end - t0);
        // the new row, if this tile and this wave have it
        const bool has_new = FUSED && t0 + tn == L;
        const int new_pass = has_new && (L - 1 - t0) % TP / TPW == wave ? (L - 1 - t0) / TP : -1;
        auto patch = [&](i32x4 &codes, int kv) {
            if (tl == (L - 1 - t0) % TP) codes = *reinterpret_cast<const i32x4 *>(&new_codes[kv][4 * (tid % (PPT * HP))]);
        };
        auto patch_scales = [&](uint32_t &sw, int kv) {
            if (has_new && t0 + scale_t == L - 1) {
                const f16 *p = &new_scales[kv][lane % HP * GPT];
                sw = GPT == 2 ? *reinterpret_cast<const uint32_t *>(p) : *reinterpret_cast<const uint16_t *>(p);
            }
        };
        patch_scales(ksw, 0);
        vsw = load_scales(vsbuf, t0);
        // ---- scores
        float mx[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) mx[r] = -INFINITY;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (u * TP + wave_t0 < tn) {                // (else the whole wave is past the end)
                const int t = u * TP + tl;
                const bool ok = t < tn;
                if (FUSED && new_pass == u) patch(slot[u], 0);
                const h2 s2 = scale_of(ksw, u);
                float dot[RC][4];           // independent chains: the dot instruction accumulates in place
#pragma unroll
                for (int r = 0; r < RC; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) dot[r][i] = 0.0f;
#pragma unroll
                for (int i2 = 0; i2 < 4; i2 += 2) {         // two dwords at a time: registers
                    h2 kh[2][4];
                    dequant(slot[u][i2], s2, kh[0]);
                    dequant(slot[u][i2 + 1], s2, kh[1]);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int i = i2; i < i2 + 2; ++i)   // channels (8 id + e, 8 id + e + 4), id = 4 piece + i
#pragma unroll
                            for (int r = 0; r < RC; ++r)
                                dot[r][i] = __builtin_amdgcn_fdot2(qr[r][4 * i + e], kh[i - i2][e], dot[r][i], false);
                }
#pragma unroll
                for (int r = 0; r < RC; ++r) {
                    float v = (dot[r][0] + dot[r][1]) + (dot[r][2] + dot[r][3]);
                    v += quad_swap<0xB1>(v);                    // lane ^ 1
                    if (PPT == 4) v += quad_swap<0x4E>(v);      // lane ^ 2
                    v *= scale;
                    if (ok && piece == 0) sc[hs * RC + r][t] = v;
                    if (ok) mx[r] = fmaxf(mx[r], v);
                }
            }
            if constexpr (VS == 1) slot[u] = load_codes(vbuf, t0 + u * TP);        // the freed slot takes V
            else load_vwords(vword[u], t0 + u * TP);
        }
#pragma unroll
        for (int r = 0; r < HP * RC; ++r) {
            const float m = wave_max(HP == 1 || hs == r ? mx[HP == 1 ? r : 0] : -INFINITY);
            if (lane == 0) wmax[r][wave] = m;
        }
        __syncthreads();                // scores and wave maxima visible
        float alpha[RC];
#pragma unroll
        for (int r = 0; r < HP * RC; ++r) {
            float tm = wmax[r][0];
#pragma unroll
            for (int w = 1; w < NW; ++w) tm = fmaxf(tm, wmax[r][w]);
            const float m_new = fmaxf(m_run[r], tm);
            const float a = __expf(m_run[r] - m_new);           // 0 on the first tile
            if (HP == 1) alpha[r] = a;
            else alpha[0] = r == 0 || hs == r ? a : alpha[0];
            m_run[r] = m_new;
            if (HP > 1 && wave / (NW / HP) != r) continue;      // 512 threads per head
            const int t = tid % DEC_THREADS;
            float sum = 0.0f;
            if (t < tn) {
                sum = __expf(sc[r][t] - m_new);
                sc[r][t] = sum;
            }
            sum = wave_sum(sum);
            if (lane == 0) wsum[r][wave % (NW / HP)] = sum;
        }
        __syncthreads();                // probabilities and wave sums visible
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            float ts = wsum[hs * RC + r][0];
#pragma unroll
            for (int w = 1; w < NW / HP; ++w) ts += wsum[hs * RC + r][w];
            l_run[r] = l_run[r] * alpha[r] + ts;
#pragma unroll
            for (int e = 0; e < VC; ++e) acc[r][e] *= alpha[r];
        }
        // ---- p * v_hat; the freed slots take the next tile's K
        patch_scales(vsw, 1);
        if (MULTI) ksw = load_scales(ksbuf, t0 + DEC_TILE);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (u * TP + wave_t0 < tn) {
                const int t = u * TP + tl;
                const bool ok = t < tn;
                if (FUSED && new_pass == u) {
                    if constexpr (VS == 1) patch(slot[u], 1);
                    else if (tl == (L - 1 - t0) % TP)
#pragma unroll
                        for (int i = 0; i < VD; ++i) vword[u][i] = new_codes[1][4 * piece + VD * vsp + i];
                }
                const h2 s2 = scale_of(vsw, u);
                float pv[RC];
#pragma unroll
                for (int r = 0; r < RC; ++r) pv[r] = ok ? sc[hs * RC + r][t] : 0.0f;
#pragma unroll
                for (int i = 0; i < VD; ++i) {
                    h2 vh[4];
                    dequant(VS == 1 ? (uint32_t)slot[u][i] : vword[VS > 1 ? u : 0][i], s2, vh);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int r = 0; r < RC; ++r) {
                            acc[r][8 * i + e] = fmaf(pv[r], (float)vh[e][0], acc[r][8 * i + e]);
                            acc[r][8 * i + e + 4] = fmaf(pv[r], (float)vh[e][1], acc[r][8 * i + e + 4]);
                        }
                }
            }
            if (MULTI) slot[u] = load_codes(kbuf, t0 + DEC_TILE + u * TP);
        }
        if (MULTI) __syncthreads();     // the tile's scores have been consumed
    }
    // ---- the token lanes meet in LDS, summed in lane order (the loop over r is unrolled to keep acc in registers)
#pragma unroll
    for (int r = 0; r < RC; ++r) {
        if (r >= nr) break;
        if (r) __syncthreads();
#pragma unroll
        for (int e = 0; e < VC; ++e) red[(DH * hs + VC * piece + e) * RROW + TPW * (PPT * hs + piece) + tl] = acc[r][e];
        if (HP > 1 && lane < PPT * HP && piece == 0) lsum[hs] = l_run[r];       // (every lane has its head's)
        __syncthreads();
        if (tid < HP * DH / VS) {
            const int hd = tid / DH, cv = tid % DH, c = VS == 1 ? cv : cv / VC * 32 + vsp * VC + cv % VC;
            float out = 0.0f;
            const float4 *rp = reinterpret_cast<const float4 *>(red + (DH * hd + cv) * RROW + TPW * (PPT * hd + cv / VC));
#pragma unroll 8
            for (int i = 0; i < TP / 4; ++i) {
                const float4 v = rp[i];
                out += v.x;
                out += v.y;
                out += v.z;
                out += v.w;
            }
            const int hq = (h + hd) * rep + r0 + r;
            const float l = HP > 1 ? lsum[hd] : l_run[r];
            if (SPLIT) {
                float *p = part + ((size_t)(b * n_kv_heads * rep + hq) * n_split + sp) * (DH + 2);
                p[c] = out;
                if (c == 0) { p[DH] = m_run[r]; p[DH + 1] = l; }
            } else {
                o[(size_t)b * d + hq * DH + c] = (f16)(out / l);
            }
        }
    }
}

// One workgroup per (sequence, query head): the splits' outputs under a common maximum.  MOST splits are loaded at once (past the last
// the last one again, unused): the launch is a round trip to memory, not one and one more for every few splits (grouped-query
// layer, 28 heads, 3 sequences of 4003 rows, 4 splits: 65.5 -> 64.5 us, one of 7990, 16 splits: 60.7 -> 53.4).
template <int DH, int MOST>
__global__ __launch_bounds__(DH) void decode_combine_kernel(const float *__restrict__ part, int n_split, f16 *__restrict__ o)
{
    const float *p = part + (size_t)blockIdx.x * n_split * (DH + 2);
    float pm[MOST], pl[MOST], po[MOST];
#pragma unroll
    for (int s = 0; s < MOST; ++s) {
        const float *ps = p + min(s, n_split - 1) * (DH + 2);
        pm[s] = ps[DH];
        pl[s] = ps[DH + 1];
        po[s] = ps[threadIdx.x];
    }
    float m = -INFINITY, l = 0.0f, out = 0.0f;
#pragma unroll
    for (int s = 0; s < MOST; ++s) m = fmaxf(m, pm[s]);
#pragma unroll
    for (int s = 0; s < MOST; ++s) {
        if (s >= n_split) break;
        const float a = __expf(pm[s] - m);          // 0 for a split without rows
        l = __builtin_fmaf(a, pl[s], l);
        out = __builtin_fmaf(a, po[s], out);
    }
    o[(size_t)blockIdx.x * DH + threadIdx.x] = (f16)(out / l);
}

template <int DH, bool FUSED>
int launch_decode(const f16 *q, int Hq, const quota_kv_cache *c, int len, f16 *o, const DecodeNew &nw, float *part,
                  hipStream_t st)
{
    const int d = Hq * DH, dkv = c->H * DH, rep = Hq / c->H, rc = rep == 1 ? 1 : 2;
    const bool stepped = c->step_dev != nullptr;
    const int longest = stepped ? c->len + c->max_steps : len;
    const double rows = (double)c->B * longest;
    ProfScope prof(QUOTA_K_ATTENTION_DECODE, 4.0 * rows * d, rows * (dkv + dkv / 16.0) + 4.0 * c->B * d, st);
    const int heads = c->H * c->B * ((rep + rc - 1) / rc);
    // two heads per workgroup where that still leaves one for every CU
    const bool pairs = rep == 1 && c->H % 2 == 0 && heads >= 2 * DEC_SPLIT_GRID;
    // as many parts as any length within the loop is split into
    int n_split = 1;
    for (int n = ((stepped ? c->len + 1 : len) + DEC_TILE - 1) / DEC_TILE; part && n <= (longest + DEC_TILE - 1) / DEC_TILE; ++n) {
        const int t = split_tiles(n, heads);
        n_split = max(n_split, (n + t - 1) / t);
    }
    const bool one_tile = longest <= DEC_TILE;
    auto run = [&](auto kernel_tag, int hp, int vs = 1) {
        constexpr auto kernel = decltype(kernel_tag)::value;
        const size_t lds = dec_red_floats(DH, hp, vs) * sizeof(float);
        if (!grant_lds<kernel>()) return QUOTA_ERR_HIP;
        kernel<<<dim3(heads * n_split * vs / hp), dim3(hp * DEC_THREADS), lds, st>>>(
            c->step_dev, nw.pos, heads * n_split * vs / hp, c->H, rep, n_split, d, dkv, q, (uint32_t *)c->k_codes, (f16 *)c->k_scales, (uint32_t *)c->v_codes,
            (f16 *)c->v_scales, c->capacity, stepped ? c->len : len, c->max_steps, heads, o, nw, part);
        QUOTA_RETURN_IF_LAUNCH_FAILED();
        return QUOTA_OK;
    };
#define KERNEL(RC, HP, MULTI, SPLIT, VS)                                                               \
    std::integral_constant<decltype(&decode_attention_kernel<DH, RC, HP, MULTI, FUSED, SPLIT, VS>),    \
                           &decode_attention_kernel<DH, RC, HP, MULTI, FUSED, SPLIT, VS>>()
    if constexpr (FUSED) {
        if (n_split > 1) {
            const int rcode = rep == 1 ? run(KERNEL(1, 1, true, true, 1), 1) : run(KERNEL(2, 1, true, true, 1), 1);
            if (rcode != QUOTA_OK) return rcode;
            static_assert(DEC_LMAX <= 16 * DEC_TILE, "");
            const auto combine = n_split <= 4 ? decode_combine_kernel<DH, 4> : n_split <= 8 ? decode_combine_kernel<DH, 8> : decode_combine_kernel<DH, 16>;
            combine<<<dim3(c->B * Hq), dim3(DH), 0, st>>>(part, n_split, o);
            QUOTA_RETURN_IF_LAUNCH_FAILED();
            return QUOTA_OK;
        }
        // V's channels by four workgroups where that leaves one for every CU (32 layers of 7B, one sequence, 640 to 122 rows 1301 -> 1259 us a step; 8
        // grouped-query layers, two sequences 453 -> 436), by two for pairs of query heads (eight sequences 518 -> 507; 7B, four: 457 -> 456)
        if (heads * 4 <= DEC_SPLIT_GRID) {
            if (rep == 1) return one_tile ? run(KERNEL(1, 1, false, false, 4), 1, 4) : run(KERNEL(1, 1, true, false, 4), 1, 4);
            return one_tile ? run(KERNEL(2, 1, false, false, 4), 1, 4) : run(KERNEL(2, 1, true, false, 4), 1, 4);
        }
        if (rep > 1 && heads * 2 <= DEC_SPLIT_GRID)
            return one_tile ? run(KERNEL(2, 1, false, false, 2), 1, 2) : run(KERNEL(2, 1, true, false, 2), 1, 2);
    }
    if (pairs) return one_tile ? run(KERNEL(1, 2, false, false, 1), 2) : run(KERNEL(1, 2, true, false, 1), 2);
    if (rep == 1) return one_tile ? run(KERNEL(1, 1, false, false, 1), 1) : run(KERNEL(1, 1, true, false, 1), 1);
    return one_tile ? run(KERNEL(2, 1, false, false, 1), 1) : run(KERNEL(2, 1, true, false, 1), 1);
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
