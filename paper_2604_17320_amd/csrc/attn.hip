// Causal prefill attention over the dequantized 4-bit K/V (fp16 MFMA, fp32
// online softmax) and the attention-cue pass of Eq. 6 (column masses).
//
// Pass 1 works on transposed tiles so that every softmax statistic is a
// per-lane scalar: S^T = K Q^T puts the query on the lane (column) and the
// keys on the accumulator registers; the probabilities then feed
// O^T += V^T P^T straight from those registers (their register->key mapping is
// the k-slot mapping chosen for the B operand of v_mfma_f32_32x32x16_f16; a
// contraction does not care which element sits in which k-slot as long as both
// operands agree, so V^T is read with the same key-to-slot mapping).
//
// Pass 2 owns key columns instead: S = Q K^T puts the key on the lane, so the
// column sums over queries are in-lane adds in a fixed order (deterministic,
// no atomics).  It needs the final log-sum-exp of every query row from pass 1.  A third, small pass takes
// the means over the heads.
//
// Both are bound by the matrix cores, the exponentials and LDS about equally (a wave's 64-key tile: 32 matrix
// instructions = 1024 cycles, 32 exponentials and 100 other vector instructions = 900), so they run two
// or more unsynchronised workgroups per SIMD and keep the rest away: tiles go from global memory to LDS without
// passing registers, double-buffered, one barrier a tile; rows are unpadded and their 16-byte pieces
// permuted so that every access spreads over all banks; V stays row-major and is transposed by the LDS read;
// the output is rescaled only when a maximum moved.  4 x 2944 tokens, 40 heads of 128: 562 us (V transposed
// by 2-byte LDS stores, tiles through registers) -> 442 us; column masses 358 -> 247 us.
#include <type_traits>
#include "common.h"
#include "internal.h"
#include "gemm_common.h"
#include "ldscopy.h"
#include "ldsgrant.h"
#include "prefetch.h"
#include "headmeans.h"

namespace {

constexpr int KT = 64;       // keys per tile (pass 1), queries per tile (pass 2)

// 2^x on the transcendental unit, without the range handling of exp2f (its extra instructions only
// matter for results below the smallest normal number, which are zero for a softmax anyway)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// A tile in LDS: KT rows of DH halves; 16-byte piece c of row r sits at piece c ^ tile_swizzle(r).  Eight rows in a
// row (a b128 read of one column of pieces) and four rows x four neighbouring pieces (a transposing read)
// each cover all banks.
template <int DH>
__device__ __forceinline__ int tile_swizzle(int r)
{
    return DH == 128 ? ((r & 3) << 2 | (r >> 2 & 3)) : ((r >> 1 & 1) << 2 | (r >> 2 & 1) << 1);
}
// Copies of KT rows of a matrix into a tile, by W waves, each its share.  A thread's places in a tile are a fixed number of
// rows apart, and their offsets are made once; rows behind the last come as zeros from the buffer's own
// bounds instead of being clamped, and a tile behind the last fetches nothing, so that its pieces need no branch and can be
// started one by one between the products.
template <int DH, int W>
struct TileCopy {
    static constexpr int CPR = DH / 8, PER = KT * CPR / (64 * W), ROWS = 64 * W / CPR;      // rows of a copy by W waves
    unsigned row_bytes, off[PER], lds_wave;
    __device__ __forceinline__ explicit TileCopy(int stride) : row_bytes(2 * stride)
    {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % W;
        const int r = wave * (64 / CPR) + lane / CPR;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            off[j] = (unsigned)(r + ROWS * j) * row_bytes + 16 * (lane % CPR ^ tile_swizzle<DH>(r + ROWS * j));
            asm volatile("" : "+v"(off[j]));
        }
        lds_wave = wave * 1024;
    }
    // The copy of rows row0 .. row0 + KT - 1 of a matrix of `rows` into the tile at lds, in PER pieces: zeros behind the last row
    struct Run {
        i32x4 buffer;
        unsigned lds;
    };
    __device__ __forceinline__ Run run(const f16 *base, int row0, int rows, unsigned lds) const
    {
        const int left = min(rows - row0, KT);
        const uint64_t at = (uint64_t)base + (uint64_t)(unsigned)row0 * row_bytes;
        return Run{i32x4{(int)(uint32_t)at, (int)(uint32_t)(at >> 32) & 0xffff, left > 0 ? (int)((left - 1) * row_bytes + 2 * DH) : 0, 0x00020000},
                   lds + lds_wave};
    }
    __device__ __forceinline__ void piece(const Run &to, int j) const
    {
        asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(to.lds + 1024 * W * j), "v"(off[j]), "s"(to.buffer) : "memory");
    }
    __device__ __forceinline__ void operator()(const f16 *base, int row0, int rows, unsigned lds) const
    {
        const Run to = run(base, row0, rows, lds);
#pragma unroll
        for (int j = 0; j < PER; ++j) piece(to, j);
    }
};
// The 16-byte pieces 2 t + hl of row r of a tile, t = 0, 1, ...: piece t is at first ^ (32 t) bytes
template <int DH>
__device__ __forceinline__ int piece_address(int r, int hl) { return r * (2 * DH) + ((hl ^ tile_swizzle<DH>(r)) << 4); }

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// the larger of a lane's value and that of the lane 32 away, without the trip through LDS of a shuffle
__device__ __forceinline__ float halves_max(float v)
{
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}

template <int DH, int W, typename PRE>
__global__ __launch_bounds__(64 * W, W / 2) void attn_fwd_kernel(
    int wgs, int N, int H, int Hkv, const f16 *__restrict__ q, const f16 *__restrict__ khat, const f16 *__restrict__ vhat, f16 *__restrict__ o,
    float scale_log2, float *__restrict__ lse2, PRE pre)
{
    if ((int)blockIdx.x >= wgs) {
        prefetch<64 * W>(pre, blockIdx.x - wgs, gridDim.x - wgs);
        return;
    }
    constexpr int T = DH / 16;       // k-steps (16 channels each) of the QK product
    constexpr int DB = DH / 32;      // 32-channel blocks of the output
    constexpr int TB = KT * DH * 2;  // bytes of a tile
    __shared__ __align__(16) char sm[2][2][TB];         // [buffer][K, V]
    // XCD-aware order: a head's workgroups, longest first, run on one XCD, whose L2 holds its K and V
    constexpr int QB = 32 * W;       // queries of a workgroup
    const int nq = (N + QB - 1) / QB, work = xcd_remap(blockIdx.x, wgs), bh = work / nq;
    const int b = bh / H, h = bh % H, q0 = (nq - 1 - work % nq) * QB;
    const int d = H * DH;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l32 = lane & 31, hl = lane >> 5;
    const int qw0 = q0 + wave * 32, qi = qw0 + l32;       // this lane's query
    const size_t base = (size_t)b * N * d + (size_t)h * DH;
    // K/V rows have Hkv heads; query head h reads K/V head h / (H / Hkv)
    const int dkv = Hkv * DH;
    const size_t kvbase = (size_t)b * N * dkv + (size_t)(h / (H / Hkv)) * DH;
    const int q_last_wg = min(q0 + QB - 1, N - 1);
    const TileCopy<DH, W> tile_copy(dkv);
    auto copy = [&](int kt0, int buf) {
        tile_copy(khat + kvbase, kt0, N, lds_address(sm[buf][0]));
        tile_copy(vhat + kvbase, kt0, N, lds_address(sm[buf][1]));
    };
    copy(0, 0);

    f16x8 qf[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
        qf[t] = *reinterpret_cast<const f16x8 *>(q + base + (size_t)min(qi, N - 1) * d + 16 * t + 8 * hl);
    f32x16 oacc[DB], zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
    asm volatile("" : "+v"(zero));           // (a register operand, instead of zeroing every accumulator)
#pragma unroll
    for (int i = 0; i < DB; ++i) oacc[i] = zero;
    float m_run = -INFINITY, l_run = 0.0f;

    const int k_at = piece_address<DH>(l32, hl);
    // V^T: lanes s of a group of 16 read 4 keys x 16 channels (lane s: key s / 4, channels 4 (s % 4) ..) and get channel s
    int v_at[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int sl = lane & 15, r = 8 * half + 4 * hl + (sl >> 2), c = 2 * (lane >> 4 & 1) + (sl >> 1 & 1);
        v_at[half] = r * (2 * DH) + ((c ^ tile_swizzle<DH>(r)) << 4) + 8 * (sl & 1);
    }
    int buf = 0;
    for (int kt0 = 0; kt0 <= q_last_wg; kt0 += KT, buf ^= 1) {
        drain();
        __syncthreads();                     // the tile is here, the other buffer has been read
        if (kt0 + KT <= q_last_wg) copy(kt0 + KT, buf ^ 1);
        if (kt0 > qw0 + 31) continue;        // tile entirely above this wave's diagonal
        const char *kt = sm[buf][0], *vt = sm[buf][1];

        f32x16 s[2];
        // (fragments a step ahead of their products, and the row maximum without LDS: they are on the wave's one chain; 640
        // tokens, 32 heads 18.5 -> 17.2 us, 4 x 2944, 40 heads 440 -> 434)
        f16x8 kf[2][2];
        auto fragments = [&](int t) {
#pragma unroll
            for (int sb = 0; sb < 2; ++sb)
                kf[t & 1][sb] = *reinterpret_cast<const f16x8 *>(kt + (k_at ^ 32 * t) + 32 * sb * (2 * DH));
        };
        fragments(0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (t + 1 < T) fragments(t + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int sb = 0; sb < 2; ++sb)
                s[sb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t & 1][sb], qf[t], t ? s[sb] : zero, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the maximum is taken on the raw logits (the scale is positive) and the scale is folded into
        // the exponent's fused multiply-add: exp2(s * scale - m), one instruction per score less
        float mx = -INFINITY;
        // only a tile that reaches this wave's diagonal or the end of the sequence needs the mask
        if (kt0 + KT - 1 > qw0 || kt0 + KT > N) {
#pragma unroll
            for (int sb = 0; sb < 2; ++sb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    int key = kt0 + 32 * sb + 8 * (r >> 2) + 4 * hl + (r & 3);
                    s[sb][r] = (key <= qi && key < N) ? s[sb][r] : -INFINITY;
                }
        }
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sb][r]);
        mx = halves_max(mx);
        float m_new = fmaxf(m_run, mx * scale_log2);
        float alpha = fast_exp2(m_run - m_new);
        m_run = m_new;
        float psum = 0.0f;
        // k-slot j of step u holds key 32 sb + 16 u + 8 (j / 4) + 4 hl + j % 4: registers 8u .. 8u+7
        f16x8 pf[2][2];
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float p[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) p[j] = fast_exp2(__builtin_fmaf(s[sb][8 * u + j], scale_log2, -m_new));
                psum += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
                pf[sb][u] = f16x8{(f16)p[0], (f16)p[1], (f16)p[2], (f16)p[3],
                                  (f16)p[4], (f16)p[5], (f16)p[6], (f16)p[7]};
            }
        l_run = l_run * alpha + psum;
        if (__ballot(alpha != 1.0f)) {       // (times one changes nothing)
#pragma unroll
            for (int i = 0; i < DB; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
        }
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < DB; ++i) {
                    const char *vb = vt + (32 * sb + 16 * u) * (2 * DH);
                    const f16x4 v0 = __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(vb + (v_at[0] ^ 64 * i))));
                    const f16x4 v1 = __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(vb + (v_at[1] ^ 64 * i))));
                    const f16x8 vf = f16x8{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                    oacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pf[sb][u], oacc[i], 0, 0, 0);
                }
    }
    float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    if (qi < N) {
        float inv = 1.0f / l_tot;
#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f16x4 ov = f16x4{(f16)(oacc[i][4 * g + 0] * inv), (f16)(oacc[i][4 * g + 1] * inv),
                                 (f16)(oacc[i][4 * g + 2] * inv), (f16)(oacc[i][4 * g + 3] * inv)};
                *reinterpret_cast<f16x4 *>(o + base + (size_t)qi * d + 32 * i + 8 * g + 4 * hl) = ov;
            }
        if (hl == 0) lse2[((size_t)b * H + h) * N + qi] = m_run + log2f(l_tot);
    }
}

// One workgroup per 32 W visual keys of a (sequence, head); wave w of a group of W owns 32 of them.
// The first key block meets every query tile, a chain that bounds launches of few workgroups: there G = 2 groups take the tiles in
// turn, each through LDS of its own, and the second's sums are added to the first's (32 heads, 165 / 400 / 640 tokens 10.3 / 15.2 / 16.6 ->
// 9.3 / 13.2 / 13.1 us, 28 heads, 1101 tokens 25.7 -> 18.9; four groups take longer below a thousand tokens).  A group alone keeps two
// pairs of sums, which its tiles add to in turn: a sequence has the same masses however many share its launch (4 x 2944 tokens,
// 40 heads 237.7 us with one pair, 239.1 so, 16 x 704 0.2 more; the two turns inlined instead of the sums exchanged: 32 x 80 tokens, 8 heads 7.1 -> 7.9).
template <int DH>
constexpr size_t colmass_lds(int G, int W) { return (size_t)G * 2 * (KT * DH * 2 + KT * 4) + (G - 1) * 32 * W * sizeof(float2); }
template <int DH, int G, int W, typename PRE>
__global__ __launch_bounds__(64 * W * G, G == 1 ? 3 : 1) void colmass_kernel(
    int wgs, int N, int H, int Hkv, int vis_begin, int Nv, const f16 *__restrict__ q, const f16 *__restrict__ khat, const float *__restrict__ lse2,
    float2 *__restrict__ partial, float scale_log2, PRE pre)
{
    if ((int)blockIdx.x >= wgs) {
        prefetch<64 * W * G>(pre, blockIdx.x - wgs, gridDim.x - wgs);
        return;
    }
    constexpr int T = DH / 16, TB = KT * DH * 2;
    extern __shared__ __align__(16) char sm[];            // [group][buffer][tile], [group][buffer][lse], [group - 1][key]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6) % W, l32 = lane & 31, hl = lane >> 5;
    const int grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / (64 * W));
    char *const sm_q = sm + grp * 2 * TB;
    float *const sm_lse = reinterpret_cast<float *>(sm + G * 2 * TB) + grp * 2 * KT;
    float2 *const sm_sum = reinterpret_cast<float2 *>(sm + G * 2 * (TB + 4 * KT));
    // XCD-aware order, as in pass 1; the first keys have the most queries
    constexpr int KB = 32 * W;       // keys of a workgroup
    const int nk = (Nv + KB - 1) / KB, work = xcd_remap(blockIdx.x, wgs), bh = work / nk, kb = work % nk;
    const int d = H * DH;
    const int b = bh / H, h = bh % H;
    const int kwg = vis_begin + kb * KB;                 // first key of the workgroup
    const int key = kwg + wave * 32 + l32;                // this lane's key column
    const bool key_ok = key < vis_begin + Nv;
    const size_t base = (size_t)b * N * d + (size_t)h * DH;
    const float *lse = lse2 + ((size_t)b * H + h) * N;

    const TileCopy<DH, W> tile_copy(d);
    auto copy = [&](int qt0, int buf) {
        tile_copy(q + base, qt0, N, lds_address(sm_q + buf * TB));
        if (wave == 0) copy4_to_lds(lse, 4 * min(qt0 + lane, N - 1), lds_address(sm_lse + buf * KT));
    };
    const int qt_first = (kwg / KT) * KT;
    if (qt_first + grp * KT < N) copy(qt_first + grp * KT, 0);
    f16x8 kf[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
        kf[t] = *reinterpret_cast<const f16x8 *>(khat + (size_t)b * N * (Hkv * DH) + (size_t)(h / (H / Hkv)) * DH +
                                                 (size_t)(key_ok ? key : N - 1) * (Hkv * DH) + 16 * t + 8 * hl);
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
    asm volatile("" : "+v"(zero));
    float acc_txt = 0.0f, acc_vis = 0.0f, other_txt = 0.0f, other_vis = 0.0f;      // G = 1: other: of the tiles before and behind this one
    auto next_sums = [&] {
        if constexpr (G == 1) {
            const float txt = acc_txt, vis = acc_vis;
            acc_txt = other_txt;
            acc_vis = other_vis;
            other_txt = txt;
            other_vis = vis;
        }
    };
    const int q_at = piece_address<DH>(l32, hl);
    int buf = 0;
    for (int qg0 = qt_first; qg0 < N; qg0 += G * KT, buf ^= 1, next_sums()) {
        drain();
        __syncthreads();
        const int qt0 = qg0 + grp * KT;
        const bool more = qt0 + G * KT < N;
        constexpr int PER = TileCopy<DH, W>::PER;             // (at the top they took the address unit all at once: 4 x 2944 tokens, 40 heads 252 -> 230 us)
        const auto next = tile_copy.run(q + base, qt0 + G * KT, N, lds_address(sm_q + (buf ^ 1) * TB));
        if (more && wave == 0) copy4_to_lds(lse, 4 * min(qt0 + G * KT + lane, N - 1), lds_address(sm_lse + (buf ^ 1) * KT));
        if (qt0 + KT - 1 < kwg + wave * 32) {             // all queries before this wave's keys
#pragma unroll
            for (int j = 0; j < PER; ++j) tile_copy.piece(next, j);
            continue;
        }
        if (G > 1 && qt0 >= N) continue;                  // (every group meets every barrier)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            f32x16 s;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (sb == 0 && t % (T / PER) == 0) tile_copy.piece(next, t / (T / PER));
                f16x8 qf = *reinterpret_cast<const f16x8 *>(sm_q + buf * TB + (q_at ^ 32 * t) + 32 * sb * (2 * DH));
                s = __builtin_amdgcn_mfma_f32_32x32x16_f16(qf, kf[t], t ? s : zero, 0, 0, 0);
            }
            // queries qb0 .. qb0 + 31; register r holds query qb0 + 8 (r / 4) + 4 hl + r % 4
            const int qb0 = qt0 + 32 * sb, vis_end = vis_begin + Nv;
            const float *ls = sm_lse + buf * KT + 32 * sb + 4 * hl;
            // the causal / end-of-sequence mask is only needed when the query block reaches this
            // wave's keys or the end of the sequence (lanes without a key accumulate values that
            // are never stored); a block of one kind of query adds to one sum
            const bool masked = qb0 < kwg + wave * 32 + 31 || qb0 + 32 > N;
            const bool all_vis = qb0 >= vis_begin && qb0 + 32 <= vis_end, all_txt = qb0 + 32 <= vis_begin || qb0 >= vis_end;
            if (!masked && (all_vis || all_txt)) {
                float a = all_vis ? acc_vis : acc_txt;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 l4 = *reinterpret_cast<const f32x4 *>(ls + 8 * r4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) a += fast_exp2(__builtin_fmaf(s[4 * r4 + e], scale_log2, -l4[e]));
                }
                if (all_vis) acc_vis = a;
                else acc_txt = a;
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int qi = qb0 + 8 * (r >> 2) + 4 * hl + (r & 3);
                    float p = fast_exp2(__builtin_fmaf(s[r], scale_log2, -ls[8 * (r >> 2) + (r & 3)]));
                    p = (key <= qi && qi < N) ? p : 0.0f;
                    bool vis = qi >= vis_begin && qi < vis_end;
                    acc_vis += vis ? p : 0.0f;
                    acc_txt += vis ? 0.0f : p;
                }
            }
        }
    }
    drain();                                              // (pieces of a tile behind the last)
    acc_txt += __shfl_xor(acc_txt, 32, 64);
    acc_vis += __shfl_xor(acc_vis, 32, 64);
    if constexpr (G > 1) {
        if (grp && hl == 0) sm_sum[(grp - 1) * KB + wave * 32 + l32] = make_float2(acc_txt, acc_vis);
        __syncthreads();
        if (grp) return;
#pragma unroll
        for (int g = 0; g < G - 1; ++g) {
            const float2 v = sm_sum[g * KB + wave * 32 + l32];
            acc_txt += v.x;
            acc_vis += v.y;
        }
    } else {
        acc_txt += other_txt + __shfl_xor(other_txt, 32, 64);
        acc_vis += other_vis + __shfl_xor(other_vis, 32, 64);
    }
    if (key_ok && hl == 0) partial[((size_t)b * H + h) * Nv + (key - vis_begin)] = make_float2(acc_txt, acc_vis);
}

// Head means of the masses, [B][H][Nv] -> [B][Nv]: 64 keys of a sequence per workgroup, a quad of lanes per key.  A launch of its own:
// left to the last workgroup of a key block in the pass above, behind a count that releases and acquires, it
// costs more (forward, cues and means: 16 x 704 tokens, 32 heads 262 us against 196; 1 x 640 34.8 against 34.2), since
// every release writes back the L2 of its XCD.  Where the masses are few a layer leaves the means to the kernel that scores them (select.hip).
__global__ __launch_bounds__(256) void colmass_reduce_kernel(
    const float2 *__restrict__ partial, int H, int Nv, float *__restrict__ cm_inter, float *__restrict__ cm_intra)
{
    const int n64 = (Nv + 63) / 64, b = blockIdx.x / n64, i = blockIdx.x % n64 * 64 + (threadIdx.x >> 2), hq = threadIdx.x & 3;
    const float invH = 1.0f / (float)H;
    const float2 sums = head_sums(partial + (size_t)b * H * Nv, H, Nv, i, hq);
    if (i < Nv && hq == 0) {
        if (cm_inter) cm_inter[(size_t)b * Nv + i] = sums.x * invH;
        if (cm_intra) cm_intra[(size_t)b * Nv + i] = sums.y * invH;
    }
}

}  // namespace

// The scratch of an attention call, at any 4-byte address: row log-sum-exp [B][H][N], per-head column masses
// [B][H][Nv] as pairs (8-byte aligned: they are stored and loaded whole).
namespace {
struct AttnWs {
    float *lse2;
    float2 *partial;
    AttnWs(void *ws, size_t rows) : lse2((float *)ws)
    {
        partial = reinterpret_cast<float2 *>((reinterpret_cast<uintptr_t>(lse2 + rows) + 7) & ~(uintptr_t)7);
    }
};
}  // namespace

extern "C" size_t quota_attention_workspace_bytes(int B, int N, int H, int dh)
{
    (void)dh;
    if (B <= 0 || N <= 0 || H <= 0) return 0;
    return (size_t)B * H * N * sizeof(float) * 3 + 8;
}

int quota_internal_attention(const void *q_f16, const void *khat_f16, const void *vhat_f16, int B,
                             int N, int H, int Hkv, int dh, int vis_begin, int Nv, void *o_f16,
                             float *cm_inter, float *cm_intra, void *ws, hipStream_t st, PrefetchList *weights,
                             quota_cue_masses *masses)
{
    if (!q_f16 || !khat_f16 || !vhat_f16 || !o_f16 || !ws) return QUOTA_ERR_NULL;
    if (B <= 0 || N < 0 || H <= 0 || Hkv <= 0 || vis_begin < 0 || Nv < 0 || vis_begin + Nv > N)
        return QUOTA_ERR_INVALID_ARG;
    if ((dh != 64 && dh != 128) || H % Hkv != 0) return QUOTA_ERR_SHAPE;
    if (!on_lds_copies(q_f16) || !on_lds_copies(khat_f16) || !on_lds_copies(vhat_f16) || (reinterpret_cast<uintptr_t>(ws) & 3))
        return QUOTA_ERR_INVALID_ARG;
    if (N == 0) return QUOTA_OK;
    const AttnWs w(ws, (size_t)B * H * N);
    float scale_log2 = 1.4426950408889634f / sqrtf((float)dh);
    const bool cues = Nv > 0 && (cm_inter || cm_intra);
    // Workgroups of two waves, 64 queries or keys each, where those of four leave many CUs without one: shorter ones start and end sooner, and a short prompt's
    // last block is half as wide.  Four and two waves, us: forward, 32 heads, 122 / 165 / 500 / 640 tokens 7.1 / 7.8 / 14.7 / 17.1, 6.3 / 7.5 / 13.7 / 17.0, 8
    // heads of 64, 80 / 640 tokens 5.2 / 11.7, 4.5 / 11.0; cues and means behind it 7.6 / 9.7 / 12.8 / 13.3 and 6.5 / 10.3, 7.5 / 9.2 / 12.1 / 12.6 and 6.0 / 9.2.
    // Beyond 160 of four they come to the same or take longer: 40 heads, 640 tokens (200) 17.6, 18.1; 2 x 300, 32 heads (192) 10.7, 11.4; cues of 28 heads,
    // 1101 tokens (224) 18.9, 20.3.  A forward launch that also fetches stays with four (a layer of 640 tokens over changing weights 148.8, 149.7 with two).
    auto waves_for = [&](int rows) { return (long)((rows + 127) / 128) * H * B <= 160 ? 2 : 4; };
    const int w1 = weights ? 4 : waves_for(N);
    const unsigned n1 = (unsigned)((N + 32 * w1 - 1) / (32 * w1)) * H * B;
    // (time by the tiles of the longest workgroup; more than 2 MB a microsecond hold its own tiles up)
    const auto s1 = weights ? weights->take(n1, 3.0f + 1.5f * (float)((N + 63) / 64), 2.0f) : PrefetchList::Share{};
    dim3 g1(n1 + s1.wgs), blk(256);
    const f16 *q = (const f16 *)q_f16, *k = (const f16 *)khat_f16, *v = (const f16 *)vhat_f16;
    const double dM = (double)B * N, dd = (double)H * dh;
    {
        ProfScope prof(QUOTA_K_ATTENTION_FWD, 4.0 * B * dd * ((double)N * (N + 1) / 2),
                       4.0 * dM * dd + 4.0 * dM * Hkv * dh, st);
        s1.run([&](auto pre) {
            auto kernel = w1 == 4 ? (dh == 128 ? attn_fwd_kernel<128, 4, decltype(pre)> : attn_fwd_kernel<64, 4, decltype(pre)>)
                                  : (dh == 128 ? attn_fwd_kernel<128, 2, decltype(pre)> : attn_fwd_kernel<64, 2, decltype(pre)>);
            kernel<<<g1, dim3(64 * w1), 0, st>>>((int)n1, N, H, Hkv, q, k, v, (f16 *)o_f16, scale_log2, w.lse2, pre);
        });
    }
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    if (cues) {
        const int w2 = waves_for(Nv);
        const unsigned four2 = (unsigned)((Nv + 127) / 128) * H * B, n2 = (unsigned)((Nv + 32 * w2 - 1) / (32 * w2)) * H * B;
        // two groups (the same sums) where every workgroup has a CU to itself, or half of one and a chain of eight tiles (2 x 640 tokens, 32 heads 18.7 -> 16.6 us, 8 x 300
        // 16.4 -> 16.5, 4 x 640 as it was)
        const bool split = four2 <= (N >= 512 ? 512u : 256u);
        const auto s2 = weights ? weights->take(four2, 3.0f + 1.1f * (float)((N + 63) / 64), 3.5f) : PrefetchList::Share{};
        // (fetching workgroups of half the width: twice as many up to 192; a layer of 640 tokens over changing weights 148.8 us, 152.4 with as many as before, one
        // of 165 113.7, 114.2 with always twice as many)
        dim3 g2(n2 + (w2 == 2 ? min(2 * s2.wgs, 192u) : s2.wgs));
        // (query, visual key) pairs under the causal mask
        const double pairs = (double)Nv * (N - vis_begin) - (double)Nv * (Nv - 1) / 2;
        ProfScope prof(QUOTA_K_ATTENTION_COLMASS, 2.0 * B * dd * pairs, 2.0 * dM * dd + 2.0 * dM * Hkv * dh, st);
        bool granted = true;
        auto launch = [&](auto dh_tag, auto groups, auto waves, auto pre) {
            constexpr int DH = decltype(dh_tag)::value, G = decltype(groups)::value, W = decltype(waves)::value;
            constexpr auto kernel = colmass_kernel<DH, G, W, decltype(pre)>;
            if ((granted = grant_lds<kernel>()))
                kernel<<<g2, dim3(64 * W * G), colmass_lds<DH>(G, W), st>>>((int)n2, N, H, Hkv, vis_begin, Nv, q, k, w.lse2, w.partial,
                                                                            scale_log2, pre);
        };
        s2.run([&](auto pre) {
            auto with_dh = [&](auto dh_tag) {
                typedef std::integral_constant<int, 2> Two;
                typedef std::integral_constant<int, 4> Four;
                if (w2 == 2) launch(dh_tag, Two(), Two(), pre);              // (160 at most: two groups)
                else if (split) launch(dh_tag, Two(), Four(), pre);
                else launch(dh_tag, std::integral_constant<int, 1>(), Four(), pre);
            };
            if (dh == 128) with_dh(std::integral_constant<int, 128>());
            else with_dh(std::integral_constant<int, 64>());
        });
        if (!granted) return QUOTA_ERR_HIP;
        QUOTA_RETURN_IF_LAUNCH_FAILED();
        if (masses) {
            *masses = {w.partial, H, cm_inter, cm_intra};
            return QUOTA_OK;
        }
        colmass_reduce_kernel<<<dim3((unsigned)((Nv + 63) / 64) * B), blk, 0, st>>>(w.partial, H, Nv, cm_inter, cm_intra);
        QUOTA_RETURN_IF_LAUNCH_FAILED();
    }
    return QUOTA_OK;
}

extern "C" int quota_attention_prefill_gqa(const void *q_f16, const void *khat_f16,
                                           const void *vhat_f16, int B, int N, int H, int Hkv, int dh,
                                           int vis_begin, int Nv, void *o_f16, float *cm_inter,
                                           float *cm_intra, void *ws, void *stream)
{
    return quota_internal_attention(q_f16, khat_f16, vhat_f16, B, N, H, Hkv, dh, vis_begin, Nv, o_f16, cm_inter, cm_intra,
                                    ws, (hipStream_t)stream, nullptr, nullptr);
}

// ---- the same call for callers that cannot allocate ---------------------------------------
// The row log-sum-exp and the per-head column masses (the two intermediates the call above keeps
// in the caller's workspace) live in a file-scope device array instead.  Host code never uses the
// array's name as an address: each device's copy is looked up once with hipGetSymbolAddress, with
// that device current, and the kernels receive the looked-up pointer like any other buffer.
// Every element the cue pass and the head mean read has been written earlier in the same call,
// so nothing needs clearing between calls.  12 bytes a row; an odd row count, which costs 4 more, is
// below the limit.
static_assert(QUOTA_ATTENTION_STATIC_MAX_ROWS % 2 == 0, "");
static __device__ __align__(256) float attn_scratch[3 * QUOTA_ATTENTION_STATIC_MAX_ROWS];

namespace {
constexpr int kMaxDevices = 64;
float *attn_scratch_ptr[kMaxDevices];      // per device, null until the first call on it
}

extern "C" int quota_attention_prefill_static(const void *q_f16, const void *khat_f16,
                                              const void *vhat_f16, int B, int N, int H, int Hkv,
                                              int dh, int vis_begin, int Nv, void *o_f16,
                                              float *cm_inter, float *cm_intra, void *stream)
{
    if (B <= 0 || N < 0 || H <= 0) return QUOTA_ERR_INVALID_ARG;
    if ((long)B * H * N > (long)QUOTA_ATTENTION_STATIC_MAX_ROWS) return QUOTA_ERR_CAPACITY;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return QUOTA_ERR_HIP;
    if (!attn_scratch_ptr[dev]) {
        float *p = nullptr;
        if (hipGetSymbolAddress((void **)&p, HIP_SYMBOL(attn_scratch)) != hipSuccess || !p)
            return QUOTA_ERR_HIP;
        attn_scratch_ptr[dev] = p;
    }
    return quota_attention_prefill_gqa(q_f16, khat_f16, vhat_f16, B, N, H, Hkv, dh, vis_begin, Nv,
                                       o_f16, cm_inter, cm_intra, attn_scratch_ptr[dev], stream);
}

extern "C" int quota_attention_prefill(const void *q_f16, const void *khat_f16,
                                       const void *vhat_f16, int B, int N, int H, int dh,
                                       int vis_begin, int Nv, void *o_f16, float *cm_inter,
                                       float *cm_intra, void *ws, void *stream)
{
    return quota_attention_prefill_gqa(q_f16, khat_f16, vhat_f16, B, N, H, H, dh, vis_begin, Nv, o_f16,
                                       cm_inter, cm_intra, ws, stream);
}
