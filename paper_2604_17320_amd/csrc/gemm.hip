// W4A4 GEMM for gfx950 on the fp6 matrix cores: y = (int4 activations) x (int4 weights)^T with an
// fp32 scale per 128-channel weight group.  ("f8" in the names is the matrix instruction's, v_mfma_..._f8f6f4.)
//
// Small integers are exact in fp6 (e2m3), and the fp32 accumulator of v_mfma_f32_16x16x128_f8f6f4 is
// exact for sums below 2^24 units, so one such instruction returns the exact integer dot product of a
// whole 128-deep group -- already as a float.  Every element needs
// y = fma(acc_g, s_g, y), group after group; against an int8 contraction, which that chain bounds, it is half as
// long (no conversion in front of the fma).
//
// fp6 operands multiply in half the time of fp8 ones (16 cycles), and fragments are a quarter smaller.  Weights: the
// bits of c + 8 in 0..15 ARE those of the e2m3 number (c + 8) / 8, so that 16 codes take 7 vector instructions
// (gemm_common.h), one more than as e4m3 bytes.  Activations are signed e2m3 numbers a / 8, made by the row quantizers.
// The weights' offset of 8 comes back out through the
// accumulator's start value, -8 / 64 * sum of the group's activation codes.  With few rows every wave makes it by
// one more MFMA per 16 rows and group, against a constant -8 / 8, whose result already lies where the C operand wants
// it; with many (quota_a6_starts) the quantizer has written it beside the rows and it comes along through LDS (all
// waves of all column tiles made the same ones).  The 2^6 of the operands' units goes into the token scale (exact).
//
// What bounds it: the issue of vector instructions.  A product holds its SIMD's issue for 8 of its 16 cycles, every other vector
// instruction for 4, whatever the number of waves, and each product brings four fmas: issued register to register with scale chain
// and unpack the products reach 51 % of the matrix rate at 8 x 4 and 8 x 2 blocks per wave, 37 to 47 at 4 x 2, 27 to 37 on
// the 32-row tiles; without the offset products the
// launches of 1100 to 11264 rows take 2 to 9 % less (fp8 operands, 11264 x 12288 x 4096: 553 -> 532 us).  With fp6 operands for
// fp8 ones bulk launches take 5 to 11 % less.  At a thousand rows and more
// the matrix cores are busy about a third of the time; on the rows of a pruned prompt for 15 to 34 % of it, and the
// waves wait for 21 to 31 % of their lives: one stage of lookahead, and a wait for all of it.
//
// Activation format inside a layer ("A6", written by the row quantizers): four rows at a time, 384 bytes per group, of row r
// 64 bytes from 64 r on -- the first four of the six dwords of each 32 channels -- and 32 from 256 + 32 r on, the other two;
// all lines that a tile reads are read whole.  G is laid out as a whole number of stages, and one more (an odd number: with a
// power of two the rows a tile reads together share one L2 channel); behind the rows, if there are
// many of them, the start values as floats, [group][row].  The public entry point takes
// packed int4 rows and converts them while staging (PACKED_INT4).
#include "common.h"
#include "internal.h"
#include "ropequant.h"
#include "gemm_common.h"
#include "ldscopy.h"

namespace {

// Lane l of a wave owns row (A) or column (B) l % 16 and the 32 channels number l / 16 of the group for
// both operands, so the order of channels inside a group cancels; it receives column l % 16, rows
// 4 (l / 16) .. + 3 of the 16 x 16 result.

// Workgroup tile (16 RT) x (16 CT NW): NW waves side by side, each with all rows and its own 16 CT
// columns, so a weight is read and unpacked by exactly one wave and never touches LDS, while activations
// and group scales are staged in LDS.
// The K loop runs in stages of CH groups: during a stage everything of the next one is set off -- weights into
// registers, the rest into the other LDS buffer -- and a stage ends with one wait for all of it and one
// barrier; nothing in between waits for memory.
//   SP: the loads are set off at the start of the stage (0) or spread over SP / 8 of its MFMAs, so that the waves
//   do not queue for the address unit all at once, nor wait at the end for what was asked for late (64 x 128 tile, 237 x 12288 x
//   4096: 23.5 us over a quarter of the stage, 20.4 over half, 21.9 over three).
//   At the start of a stage they are left out past the last one, a round trip that the launch would wait for (32 x 64 tile, 42 x 512 x 512
//   3.72 -> 3.63 us, 165 x 9728 x 896 7.9 -> 6.8, 320 x 5632 x 1024 7.8 -> 6.8); a branch around every spread load costs longer rows more
//   than it saves short ones (38 groups in stages of 8: 7.7 -> 8.6).
// A group in LDS: the rows' 64-byte parts, then their 32-byte parts.  Lane (row c, channels 32 q ..) reads 16 bytes of the first
// and 8 of the second; 16-byte piece q of row r's first part sits at q ^ {0, 2, 3, 1}[r / 4 % 4], and the halves of the second
// are swapped in rows 8 to 15 of 16, so that the lanes of a read do not share banks.
enum ActFormat { A6, A6_STARTS, PACKED_INT4 };
enum Epilogue { PLAIN, QKV_ROPE_KV, SILU_MUL, PLAIN_PICKED };     // PICKED: of rows picked through indices
// What some launches take besides, by their epilogue (QKV_ROPE_KV, PLAIN_PICKED).  One place for both: every argument costs the
// host time.
union GemmMore {
    quota_qkv_epilogue qkv;
    quota_kept_rows kept;
};
template <int RT, int CT, int NW, int CH, int SP, ActFormat ACTS, bool ACC_OUT, Epilogue EPI>
__device__ __forceinline__ void w4a4_tile(
    const uint8_t *__restrict__ qa, const float *__restrict__ sa, int M, int K, int G,
    const uint4 *__restrict__ wp, const f16 *__restrict__ sw, int N, f16 *__restrict__ y, int ldy,
    const f16 *__restrict__ res, int ldr, int32_t *__restrict__ acc_out, int tiles_m, int tiles_n, const GemmMore &more)
{
    const quota_qkv_epilogue &qe = more.qkv;
    constexpr int NT = 64 * NW, BM = 16 * RT, WN = 16 * CT, BN = NW * WN, T = RT * CT;
    constexpr bool PACKED = ACTS == PACKED_INT4, STARTS = ACTS == A6_STARTS, QKV = EPI == QKV_ROPE_KV, SILU = EPI == SILU_MUL;
    static_assert(!SILU || (CT % 2 == 0 && !ACC_OUT), "as many blocks of gate as of up columns");
    constexpr int LA = PACKED ? (BM * 4 + NT - 1) / NT : 0;              // PACKED: 16-byte pieces per thread and group
    // else wave-wide copies of 16 bytes a lane, per wave and stage: of first parts (16 rows each) and of second ones (32 rows)
    constexpr int MC = PACKED ? 0 : CH * BM / 16 / NW, TC = PACKED ? 0 : CH * BM / 32 / NW;
    // dwords per stage, 64 to a copy: the group scales, then (STARTS) the rows' start values
    constexpr int SCOPY = CH * BN / 128, ICOPY = STARTS ? CH * BM / 64 : 0, KD = (SCOPY + ICOPY + NW - 1) / NW;
    static_assert(RT % 2 == 0 && (PACKED || CH * BM % (32 * NW) == 0) && (!STARTS || CH * BM % 64 == 0) && CH * BN % 128 == 0,
                  "whole rows per copy, whole copies of dwords, fragment double buffer");
    // one stage in LDS (in uint4): CH groups of activations (+ a spare piece for PACKED threads without one),
    // then the dwords, up to whole waves
    constexpr int AST = BM * 6 + (PACKED ? 2 : 0), GST = CH * AST, STG = GST + KD * NT / 4;
    constexpr int TROW = BN + 8, FROW = BN + 4;                          // staged output rows: fp16 (QKV), fp32
    constexpr int LDS_A = 2 * STG, LDS_Q = QKV || SILU ? 32 * TROW / 8 : 32 * FROW / 4;
    __shared__ uint4 lds_raw[LDS_A > LDS_Q ? LDS_A : LDS_Q];
    __shared__ __align__(16) float row_scale[BM];        // for the epilogue: token scales, with the 2^6 of the operands' units
    __shared__ int row_pos[QKV ? BM : 1];                // and rows of the angle tables
    const unsigned lds0 = lds_address(lds_raw);

    int tile_m, tile_n;
    tile_of(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, tile_m, tile_n);
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Token scale and position of row tid of the tile: a layer's are asked for beside the first stage, packed rows' in front (33 x 4096 x 11008: 31.6 us, 33.7 beside).
    // A layer's in front, where a stage's loads are spread, over scales that the caches hold: QKV 165 x 12288 x 4096 20.4 us, 20.0 beside, gate/up 165 x 22016 x 4096 23.7,
    // 23.45, with start values 1500 x 4096 x 11008 65.8, 65.5; plain rows without them 300 x 3584 x 18944 54.4, 54.9, 400 x 4096 x 11008 32.6, 33.0, 122 x 4096 x 4096
    // 7.12, 7.25.  But in a layer the quantizer has just written the scales: there O and down of 288 rows take 20.4 us either way, and with all four
    // projections so a stack of 32 layers 0.5 % longer.
    constexpr bool AT_ONCE = !SP && !PACKED;             // a stage's loads go out all at once
    // PICKS: row m of activations and residual is row row_src[m] of the tensors handed in.  The indices are asked for ahead of the first
    // weights and looked up behind them.  (An instantiation of its own: with the table of rows in all
    // PLAIN launches those that pick none took a barrier and a trip to LDS before their first activations: 122 x 4096 x 4096 7.39 us, 7.25 so, 256 x 4096 x 11008
    // 23.4, 23.0, 64 x 5120 x 5120 10.8, 10.4.)
    constexpr bool PICKS = EPI == PLAIN_PICKED, ADDS = EPI == PLAIN || PICKS;
    static_assert(!PICKS || (ACTS == A6 && !ACC_OUT), "(the layer's output projection)");
    __shared__ int row_src[PICKS ? BM : 1];
    const quota_kept_rows &kept = more.kept;
    int pick_j = 0, pick_b = 0, pick = 0;
    if constexpr (PICKS) {
        const int m = min(m0 + min(tid, BM - 1), M - 1);
        pick_b = m / kept.n_keep;
        pick_j = m - pick_b * kept.n_keep;
        pick = kept.index(pick_b, pick_j);
    }
    if constexpr (PACKED) {
        if (tid < BM) {
            const int m = min(m0 + tid, M - 1);
            row_scale[tid] = sa[m] * F6_UNIT;
            if constexpr (QKV) row_pos[tid] = min(max(qe.pos[m], 0), qe.n_pos - 1);
        }
    }

    // Global loads are unconditional with clamped addresses: rows past M and columns past N repeat the last
    // ones and are never stored; groups past G repeat the last one and are not used.
    const int Kb = K >> 1, fours = (M + 3) >> 2;         // PACKED: bytes per row; A6: fours of rows, bytes of one
    const unsigned four_bytes = (unsigned)quota_a6_groups(G) * 384u;
    constexpr int BB = BM / 16, TB = BM / 32;            // copies of a group's first parts, of its second ones
    // where the 16-byte piece of channels 32 p .. of a row's first part lies among four
    auto piece_of = [](int p, int row) { return p ^ (0x1320 >> (row & 12) & 3); };
    unsigned oa[PACKED ? LA : 1], om = 0, ot = 0;        // byte offsets of this thread's pieces, in group 0 or (A6) a group
    unsigned om2 = 0, dm = 0, dt = 0;                    // ... and where its wave's pieces go in LDS
    // (96 rows: the blocks that a wave copies come round in threes, and change groups in between)
    constexpr bool THREES = BB % NW != 0 && NW % BB != 0;
    unsigned om3[THREES ? 3 : 1], ot3[THREES ? 3 : 1];
    int la[LA ? LA : 1], lt[LA ? LA : 1], pa[LA ? LA : 1];       // PACKED: LDS slots (16 bytes, 8 bytes) of the piece
    // (threads without one write a spare slot: a branch would let the compiler sink the scale chain behind it)
    if constexpr (PACKED) {
#pragma unroll
        for (int j = 0; j < LA; ++j) {
            const int i = tid + NT * j, row = i >> 2, p = i & 3;
            oa[j] = (unsigned)(min(m0 + min(row, BM - 1), M - 1) - m0) * (unsigned)Kb;
            pa[j] = 16 * p;
            la[j] = row < BM ? row * 4 + piece_of(p, row) : BM * 6;
            lt[j] = row < BM ? BM * 8 + row * 4 + ((p >> 1 ^ (row >> 3 & 1)) << 1) + (p & 1) : BM * 12 + 2;
        }
    }
    // SILU: columns are gate | up, F = N / 2 of each, and a tile takes BN / 2 of either: a wave's first CT / 2 blocks are gate
    // columns, the others up columns of the same channels.
    constexpr int WC = SILU ? WN / 2 : WN, BC = SILU ? BN / 2 : BN, CB = WC / 16;       // neighbouring columns of a wave, of a tile
    const int NC = SILU ? N >> 1 : N, nc0 = tile_n * BC;
    const int nw = min(nc0 + wave * WC, NC - WC);        // this wave's first column (N is a multiple of 64)
    const bool n_ok = n0 + wave * WN < N;
    // this lane's uint4 of a wave's first 16-column block, and of its first block of up columns
    const unsigned wl = (unsigned)(c16 * 4 + q), wl_up = wl + (unsigned)NC * 4;
    // dword tid + NT k of a stage: the scales of two neighbouring columns, or the start value of a row, in one of its groups
    const float *starts = reinterpret_cast<const float *>(qa + (size_t)fours * four_bytes);
    constexpr bool ONE_GROUP = BN / 2 % 64 == 0 && (!STARTS || BM % 64 == 0);            // a wave's dwords are of one group
    unsigned os[KD];
    int gs[KD];
#pragma unroll
    for (int k = 0; k < KD; ++k) {
        const bool scale = !STARTS || wave + NW * k < SCOPY;
        const int d = scale ? min(tid + NT * k, CH * BN / 2 - 1) : min(tid + NT * k - 64 * SCOPY, CH * BM - 1);
        gs[k] = scale ? d / (BN / 2) : d / BM;
        if (ONE_GROUP) gs[k] = __builtin_amdgcn_readfirstlane(gs[k]);
        int pair = d % (BN / 2), first = 0;              // pair of columns: in its run of neighbouring ones, and the run's first
        if (SILU) {
            first = pair / (WC / 2) % 2 * (NC >> 1);
            pair = pair / WC * (WC / 2) + pair % (WC / 2);
        }
        os[k] = 4u * (unsigned)(scale ? first + min((nc0 >> 1) + pair, (NC >> 1) - 1) : min(m0 + d % BM, M - 1));
    }

    // Register sets of packed weights = stages per loop body.  With 8 x 4 blocks there is room for one: a group's weights are
    // asked for when those of the same place in the last stage have been unpacked, the second group's last of all.
    constexpr int WS = CH > 1 && T < 32 ? 2 : 1;
    constexpr bool LATE = CH > 1 && WS == 1;
    uint4 rw[WS][CH][CT];
    i32x4 ra[CH][LA ? LA : 1];                           // PACKED staging (struct uint4 here would live in scratch memory)
    // What a stage needs, load by load: for each of its groups CT weight pieces and (PACKED) LA activation pieces, then
    // the wave's copies of activations, then KD dwords.  The weights' pointer (uniform, of the next group to load) stops at the
    // last group, the activations' at the last stage (whose groups past G are in memory): what lies past them is loaded
    // but never used.  Scalar instructions count: a wave issues one of any kind at a time.
    constexpr int SPAN = SP ? CH * T * SP / 8 : 1;        // products that the loads are spread over
    constexpr int LG = CT + LA, LC = CH * LG + MC + TC, LOADS = LC + KD;
    const uint4 *wnext = wp + (size_t)nw * 4;
    const unsigned wstep = (unsigned)N * 64u;
    const uint8_t *a0 = PACKED ? qa + (size_t)m0 * Kb : PICKS ? qa : qa + (size_t)(m0 >> 2) * four_bytes;
    int gstage = 0;                                       // first group of the stage being loaded
    static_assert(!LATE || (CH == 2 && SP && (LOADS - LG) * SPAN / LOADS >= T), "the first group's products cover what comes before");
    auto load = [&](int at, int set, int half) {
        const unsigned to = (unsigned)half * (STG * 16);
        const int k = !LATE || at < LG ? at : at < LOADS - LG ? at + LG : at - (LOADS - 2 * LG);
        if (k < CH * LG) {
            const int c = k / LG, r = k % LG;
            if (r < CT) {
                rw[set][c][r] = wnext[(r < CB ? wl : wl_up) + 64 * (r % CB)];
            } else if constexpr (PACKED) {
                const unsigned kb = (unsigned)min(min(gstage + c, G - 1) * 64 + pa[r - CT], Kb - 16);
                ra[c][r - CT] = *reinterpret_cast<const i32x4 *>(a0 + (oa[r - CT] + kb));
            }
            if (r == LG - 1) wnext = (const uint4 *)((const char *)wnext + (G - gstage > c + 1 ? wstep : 0u));
        } else if (k < LC) {
            const int j = k - CH * LG;
            if constexpr (THREES) {
                const bool first = j < MC;
                const int i = first ? j : j - MC, n = first ? BB : TB, blk = wave + NW * i, c = blk / n, b = blk % n;
                copy16_to_lds(a0 + c * 384, first ? om3[i % 3] : ot3[i % 3],
                              lds0 + (to + (unsigned)(c * (AST * 16) + b * 1024 + (first ? 0 : BM * 64))));
            } else if (j < MC) {                                // block wave + NW j of the stage's, BB to a group
                const int c = BB >= NW ? j * NW / BB : j * (NW / BB), b = BB >= NW ? j * NW % BB : 0;
                copy16_to_lds(a0 + c * 384, BB > NW && j % 2 ? om2 : om, dm + (to + (unsigned)(c * AST * 16 + b * 1024)));
            } else {
                const int c = (j - MC) * (NW / TB);
                copy16_to_lds(a0 + c * 384, ot, dt + (to + (unsigned)(c * AST * 16)));
            }
        } else {
            const int j = k - LC;
            const bool scale = !STARTS || wave + NW * j < SCOPY;
            const unsigned g = (unsigned)min(gstage + gs[j], G - 1), row = (unsigned)(scale ? 2 * N : 4 * M);
            const char *base = scale ? (const char *)sw : (const char *)starts;
            copy4_to_lds(ONE_GROUP ? base + (size_t)g * row : base, ONE_GROUP ? os[j] : os[j] + g * row,
                         lds0 + (to + (unsigned)(GST * 16 + (wave + NW * j) * 256)));
        }
    };
    auto store_packed = [&](int half) {                  // convert and store what the loads brought
        if constexpr (PACKED) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                uint4 *dst = lds_raw + half * STG + c * AST;
#pragma unroll
                for (int j = 0; j < LA; ++j) {
                    uint32_t e[6];
                    codes_e2m3(ra[c][j], e);
                    dst[la[j]] = make_uint4(e[0], e[1], e[2], e[3]);
                    reinterpret_cast<uint2 *>(dst)[lt[j]] = make_uint2(e[4], e[5]);
                }
            }
        }
    };

    float yacc[RT][CT][4];
    int tot[ACC_OUT ? RT : 1][ACC_OUT ? CT : 1][4];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                yacc[i][j][r] = 0.0f;
                if (ACC_OUT) tot[i][j][r] = 0;
            }
    uint32_t flip[3];
    e2m3_flips(flip);
    // this lane's activation fragment of row block i of the group at `gp`, the start values of its four
    // results, and the scale of its column in block j
    const int fr = c16 * 4 + piece_of(q, c16), ft = c16 * 4 + ((q >> 1 ^ c16 >> 3) << 1) + (q & 1);
    i32x8 minus8 = i32x8{(int)0x28A28A28, (int)0x8A28A28A, (int)0xA28A28A2, (int)0x28A28A28, (int)0x8A28A28A, (int)0xA28A28A2, 0, 0};
    if (!STARTS) asm("" : "+v"(minus8));       // (held, not made anew for every group)
    auto read_a = [&](const uint4 *gp, int i, i32x8 &fa) {
        const uint4 a0 = gp[i * 64 + fr];
        const uint2 a1 = reinterpret_cast<const uint2 *>(gp + BM * 4)[i * 64 + ft];
        fa = i32x8{(int)a0.x, (int)a0.y, (int)a0.z, (int)a0.w, (int)a1.x, (int)a1.y, 0, 0};
    };
    // the start values of row block i's results in group c of the stage
    auto start_of = [&](const uint4 *sp, int c, int i, const i32x8 &fa) {
        if constexpr (!STARTS) return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa, minus8, f32x4{0, 0, 0, 0}, 2, 2, 0, 0, 0, 0);
        else return *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(sp + GST) + 64 * SCOPY + c * BM + 16 * i + 4 * q);
    };
    auto read_scale = [&](const uint4 *sp, int c, int j) {
        float s = (float)reinterpret_cast<const f16 *>(sp + GST)[c * BN + wave * WN + 16 * j + c16];
        asm("" : "+v"(s));           // (converted once: multiply-adds that take the half itself issue a third slower)
        return s;
    };
    // The group scale of a result is applied LAG results later, so that the matrix core's latency is
    // covered; the last ones of a group are finished during the next.  (One covers a 16-cycle product; two take as long
    // and five registers more, which the 128 x 128 tile does not have.)
    constexpr int LAG = 1;
    static_assert(T % LAG == 0, "the carried results keep their order");
    f32x4 pend[LAG];
    float pscale[LAG];
#pragma unroll
    for (int i = 0; i < LAG; ++i) { pend[i] = f32x4{0, 0, 0, 0}; pscale[i] = 0.0f; }
    auto scale_in = [&](int t, const f32x4 &a, float s) {
        const int i = t / CT, j = t % CT;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            yacc[i][j][r] = __builtin_fmaf(a[r], s, yacc[i][j][r]);
            if (ACC_OUT) tot[i][j][r] += (int)(a[r] * F6_UNIT);
        }
    };

    // A wave's priority rises with every quarter of a stage's row blocks and falls at its end, so that of two workgroups of
    // a CU the one that is ahead finishes its products while the other waits, unpacks or reads: with equal ones they fall into
    // step, multiply together and wait together (237 x 4096 x 11008 25.6 -> 23.4 us, 160 x 22016 x 4096 28.0 -> 26.0, 1280 x
    // 4096 x 11008 64.1 -> 61.2, 5808 x 22016 x 4096 400 -> 396; lowest at products, highest around the barrier: nothing).
    static_assert(CH >= 4 ? CH % 4 == 0 : RT % (4 / CH) == 0, "whole row blocks, or groups, per quarter");
    // The first weights go out as soon as their address is there, ahead of the copies' addresses and of what the epilogue needs.
    constexpr int WEIGHTS_FIRST = PACKED ? 0 : LATE ? LG : CH * LG;
#pragma unroll
    for (int k = 0; k < WEIGHTS_FIRST; ++k) load(k, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!PACKED) {
        // A copy of first parts: lane l brings row l / 4 of 16 to piece l % 4; of second ones: row l / 2 of 32 to half l % 2
        static_assert(THREES ? BB == 6 && NW == 4 : BB <= 2 * NW && (TB % NW == 0 || NW % TB == 0), "blocks of rows by wave");
        const int last = fours - 1 - (m0 >> 2), row = lane >> 2, row2 = lane >> 1;
        if constexpr (PICKS) {               // where its rows lie
            if (tid < BM) row_src[tid] = pick_b * kept.N + kept.row(pick_j, pick);
            __syncthreads();
        }
        auto first = [&](int blk) {
            const int r4 = min(4 * (blk % BB) + (row >> 2), last);
            const unsigned src = PICKS ? row_src[16 * (blk % BB) + row] : 4 * r4 + (row & 3);
            return (src >> 2) * four_bytes + (src & 3) * 64 + 16 * piece_of(lane & 3, row);
        };
        auto second = [&](int blk) {
            const int r4 = min(8 * (blk % TB) + (row2 >> 2), last);
            const unsigned src = PICKS ? row_src[32 * (blk % TB) + row2] : 4 * r4 + (row2 & 3);
            return (src >> 2) * four_bytes + 256 + (src & 3) * 32 + 16 * ((lane ^ row2 >> 3) & 1);
        };
        om = first(wave) + wave / BB % NW * 384;
        if (BB > NW) om2 = first(wave + NW);
        ot = second(wave) + wave / TB % NW * 384;
        dm = lds0 + wave / BB % NW * (AST * 16) + wave % BB * 1024;
        dt = lds0 + wave / TB % NW * (AST * 16) + BM * 64 + wave % TB * 1024;
        if constexpr (THREES) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                om3[j] = first(wave + NW * j);
                ot3[j] = second(wave + NW * j);
            }
        }
        const int m = PICKS ? row_src[min(tid, BM - 1)] : min(m0 + min(tid, BM - 1), M - 1);
        float scale = sa[m];
        int pos = 0;
        if constexpr (QKV) pos = qe.pos[m];
#pragma unroll
        for (int k = WEIGHTS_FIRST; k < LOADS; ++k) load(k, 0, 0);
        asm volatile("" : "+v"(scale), "+v"(pos));       // (asked for here, not behind the wait)
        // (the first touch of the epilogue's arguments comes from far away: here, not behind the main loop)
        if constexpr (QKV) asm volatile("" ::"s"(qe.v_scales));
        drain();
        if (tid < BM) {
            row_scale[tid] = scale * F6_UNIT;
            if constexpr (QKV) row_pos[tid] = min(max(pos, 0), qe.n_pos - 1);
        }
    } else {
#pragma unroll
        for (int k = 0; k < LOADS; ++k) load(k, 0, 0);
        drain();
    }
    // The first stage's weights are here before the barrier: left alone the compiler starts them behind it, and the waits for them, which it puts into
    // the loop and counts without the copies, wait there for loads of the next stage that have just been started (64 x 128 tile, 1101 x 3584 x
    // 18944: main loop 113900 -> 111400 cycles; 128 x 128, 1700 x 4096 x 4096 29.5 -> 28.5 us, 640 x 12288 x 4096 35.0 -> 34.4; the 32-row tiles as before).
    if constexpr (!ACC_OUT) {
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int j = 0; j < CT; ++j)
                asm volatile("" : "+v"(rw[0][c][j].x), "+v"(rw[0][c][j].y), "+v"(rw[0][c][j].z), "+v"(rw[0][c][j].w));
    }
    store_packed(0);
    __syncthreads();

    // What the epilogue needs from memory for 32 rows (round ib): a thread has row RPI * k + row0 of them, and 8 channels.  Asked for round by round,
    // each waited for memory.  The residual rows of tiles of one round come a main loop ahead (100 x 3584 x 18944 28.35 -> 28.11 us, 80 x 512 x 512
    // 3.11 -> 3.04), except of packed rows, whose 32 x 128 tile the registers would cost one of three workgroups per CU (450 x 3584 x 18944 73.1 -> 75.0).
    // Else all rounds' are asked for in front of the epilogue, and the angles a round ahead (300 x 12288 x 4096 23.3 -> 23.1).  Angles held through the
    // main loop, 16 registers a row, take a workgroup per CU from 32 x 128 (three) and 32 x 64 (five) and give nothing where there is room (1400 x 1536 x
    // 512 9.6 us, 7.8 without, 100 x 6144 x 2048 7.2, 6.9).
    constexpr int RPI = NT / (BN / 8), KI = 32 / RPI, ROUNDS = RT / 2, AR = !QKV ? 1 : KI <= 2 && ROUNDS > 1 ? 2 : 1;
    const int row0 = tid / (BN / 8), c8 = tid % (BN / 8), n8 = n0 + 8 * c8;
    float cs[AR][QKV ? KI : 1][8], sn[AR][QKV ? KI : 1][8];
    f16x8 rv[ADDS ? ROUNDS : 1][ADDS ? KI : 1];
    // (The address passes the assembly as a number and is one of global memory again behind it: loads of an address of unknown memory count as LDS
    // reads too, and in the 32-row tiles, which ask ahead of the main loop, every wait for LDS in the first stage of its body was a wait for all of
    // them: 237 x 4096 x 4096 9.4 -> 9.2 us, 80 x 1024 x 1024 4.0 -> 3.8.)
    typedef const __attribute__((address_space(1))) f16x8_at2 *global_f16x8;
    uint64_t res_at = (uint64_t)res;
    asm volatile("" : "+s"(res_at));         // (else the loads sink to where they are used)
    auto ask_angles = [&](int ib) {
        const int half = qe.dh >> 4;         // chunks per half head (4 or 8)
        if (n0 < qe.d + qe.dkv) {
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                const unsigned at = (unsigned)(row_pos[32 * ib + RPI * k + row0] * 8 * half + 8 * (c8 & (half - 1)));
                float *cp = cs[ib % AR][k], *sp = sn[ib % AR][k];
                *reinterpret_cast<float4 *>(cp) = *reinterpret_cast<const float4 *>(qe.cosT + at);
                *reinterpret_cast<float4 *>(cp + 4) = *reinterpret_cast<const float4 *>(qe.cosT + at + 4);
                *reinterpret_cast<float4 *>(sp) = *reinterpret_cast<const float4 *>(qe.sinT + at);
                *reinterpret_cast<float4 *>(sp + 4) = *reinterpret_cast<const float4 *>(qe.sinT + at + 4);
            }
        }
    };
    auto ask_residual = [&](int ib) {
        if (res && n8 < N) {
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                const int m = 32 * ib + RPI * k + row0;
                rv[ib][k] = *(global_f16x8)(res_at + 2 * ((size_t)(PICKS ? row_src[m] : min(m0 + m, M - 1)) * ldr + n8));
            }
        }
    };
    constexpr bool AHEAD = ADDS && ROUNDS == 1 && !PACKED;
    if constexpr (AHEAD) ask_residual(0);

    i32x8 fb[CT];
    const int stages = (G + CH - 1) / CH;
    i32x8 fa[2];
#pragma unroll 1
    for (int st0 = 0; st0 < stages; st0 += WS) {
#pragma unroll
        for (int su = 0; su < WS; ++su) {
            const int g0 = (st0 + su) * CH, half = WS == 2 ? su : st0 & 1, set = su;
            if (su && g0 >= G) break;
            const uint4 *sp = lds_raw + half * STG;
            read_a(sp, 0, fa[0]);
            if (CH == 1) {
#pragma unroll
                for (int j = 0; j < CT; ++j) weights_e2m3(rw[0][0][j], flip, fb[j]);
            }
            gstage = g0 + CH;
            if (!PACKED) a0 += gstage < G ? CH * 384 : 0;
            if (!AT_ONCE || gstage < G) {
#pragma unroll
                for (int k = 0; k < (SP ? 0 : LOADS); ++k) load(k, (set + 1) % WS, half ^ 1);
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (c && g0 + c >= G) break;             // uniform: the last stage may hold fewer groups
                const uint4 *gp = sp + c * AST;
                if (CH >= 4 && c == CH / 4) __builtin_amdgcn_s_setprio(1);
                if (CH >= 2 && c == CH / 2) __builtin_amdgcn_s_setprio(2);
                if (CH >= 4 && c == 3 * CH / 4) __builtin_amdgcn_s_setprio(3);
                float sc[CT];
#pragma unroll
                for (int j = 0; j < CT; ++j) sc[j] = read_scale(sp, c, j);
                if (CH > 1) {
#pragma unroll
                    for (int j = 0; j < CT; ++j) weights_e2m3(rw[set][c][j], flip, fb[j]);
                }
                // The issue order is pinned result by result (left alone the scheduler puts the scale chain
                // of a result right behind its own MFMA and waits out the matrix core's latency, and reads
                // every row block's fragments up front, which does not fit the registers): one MFMA, the
                // chain of the result LAG places back.  The next row block's fragments are read at the start of
                // a row block.
                f32x4 k4[2];
                k4[0] = start_of(sp, c, 0, fa[0]);
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    if (i + 1 < RT) read_a(gp, i + 1, fa[(i + 1) & 1]);
                    else if (c + 1 < CH) read_a(gp + AST, 0, fa[0]);
                    if (STARTS && i + 1 < RT) k4[(i + 1) & 1] = start_of(sp, c, i + 1, fa[0]);
                    if ((CH == 1 && i == RT / 4) || (CH == 2 && c == 0 && i == RT / 2)) __builtin_amdgcn_s_setprio(1);
                    if (CH == 1 && i == RT / 2) __builtin_amdgcn_s_setprio(2);
                    if ((CH == 1 && i == 3 * RT / 4) || (CH == 2 && c == 1 && i == RT / 2)) __builtin_amdgcn_s_setprio(3);
#pragma unroll
                    for (int j = 0; j < CT; ++j) {
                        __builtin_amdgcn_sched_barrier(0);
                        const int t = i * CT + j;
                        const f32x4 a = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[i & 1], fb[j], k4[i & 1], 2, 2, 0, 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (t < LAG) scale_in(T - LAG + t, pend[t], pscale[t]);
                        else scale_in(t - LAG, pend[t % LAG], sc[(t - LAG) % CT]);
                        pend[t % LAG] = a;
                        if (!STARTS && j == CT - 1 && i + 1 < RT) k4[(i + 1) & 1] = start_of(sp, c, i + 1, fa[(i + 1) & 1]);
#pragma unroll
                        for (int e = 0; e < (SP ? (LOADS - 1) / SPAN + 1 : 0); ++e) {
                            const int k = ((c * T + t) * LOADS + SPAN - 1) / SPAN + e;
                            if (k < LOADS && k * SPAN / LOADS == c * T + t) load(k, (set + 1) % WS, half ^ 1);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < LAG; ++i) pscale[i] = sc[(T - LAG + i) % CT];
            }
            __builtin_amdgcn_s_setprio(0);
            drain();
            if constexpr (LATE) {                        // (else the compiler waits for them in the middle of the next stage)
#pragma unroll
                for (int j = 0; j < CT; ++j) asm("" : "+v"(rw[0][CH - 1][j].x), "+v"(rw[0][CH - 1][j].y), "+v"(rw[0][CH - 1][j].z), "+v"(rw[0][CH - 1][j].w));
            }
            store_packed(half ^ 1);
            __syncthreads();
        }
    }
#pragma unroll
    for (int i = 0; i < LAG; ++i) scale_in(T - LAG + i, pend[i], pscale[i]);

    // epilogue: token scale (with the 2^6 of the operands' units), residual, fp16
    if constexpr (QKV) {
        // Fused epilogue of the QKV projection: 32 rows of the fp16 tile (whole heads: the tile width divides
        // the model width and is a multiple of the head size) at a time are staged in LDS by all waves; then
        // every thread takes (row, 8-channel chunk) items, of one chunk, and applies RoPE at the token's position id (q
        // and k tiles) and the 4-bit K/V group quantizer (k and v tiles) exactly as the stand-alone kernel
        // does.  q | k | v are column ranges [0,d) [d,d+dkv) [d+dkv,d+2dkv), so a tile lies in one of them.
        const MixMul mul;
        f16 *stage = reinterpret_cast<f16 *>(lds_raw);
        const int d = qe.d, dkv = qe.dkv;
        const int region = n0 < d ? 0 : (n0 < d + dkv ? 1 : 2);          // tile-uniform
        const int half = qe.dh >> 4, c = c8;                             // chunks per half head (4 or 8)
        const bool second = c & half;
        const int width = region == 0 ? d : dkv, col = n0 - (region == 0 ? 0 : (region == 1 ? d : d + dkv)) + 8 * c;
        f16 *out16 = (region == 0 ? qe.q_rot : region == 1 ? qe.khat : qe.vhat) + (size_t)m0 * width + col;
        uint32_t *codes = (region == 1 ? qe.k_codes : qe.v_codes) + (((size_t)m0 * width + col) >> 3);
        f16 *scales = (region == 1 ? qe.k_scales : qe.v_scales) + (((size_t)m0 * width + col) >> 6);
#pragma unroll
        for (int ib = 0; ib < RT / 2; ++ib) {
            if (AR > 1 && ib + 1 < ROUNDS) {          // (a round ahead; of 128 x 256 the registers hold one)
                if (ib == 0) ask_angles(0);
                ask_angles(ib + 1);
            } else if (AR == 1) {
                ask_angles(ib);
            }
            if (ib) __syncthreads();                  // the previous 32 rows have been read
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 sam = *reinterpret_cast<const f32x4 *>(row_scale + 32 * ib + 16 * h + 4 * q);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    f16 *p = stage + (16 * h + 4 * q + r) * TROW + wave * WN + c16;
#pragma unroll
                    for (int j = 0; j < CT; ++j) p[16 * j] = to_f16(yacc[2 * ib + h][j][r] * sam[r]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KI; ++k) {
                const int row = RPI * k + row0, m = 32 * ib + row;       // in the 32 rows, in the tile
                const bool m_ok = m0 + m < M;
                Pack16 x, xp, out;
                x.u = *reinterpret_cast<const uint4 *>(stage + row * TROW + 8 * c);
                if (y && m_ok) *reinterpret_cast<uint4 *>(y + (size_t)(m0 + m) * ldy + n0 + 8 * c) = x.u;
                out = x;
                if (region < 2) {
                    xp.u = *reinterpret_cast<const uint4 *>(stage + row * TROW + 8 * (c ^ half));
                    rope8(x, xp, cs[ib % AR][k], sn[ib % AR][k], second, out, mul);
                }
                const unsigned at = (unsigned)(m * width);               // elements from the tile's first row
                if (region == 0) {
                    if (m_ok) *reinterpret_cast<uint4 *>(out16 + at) = out.u;
                } else {
                    Pack16 hat;
                    f16 sc8;
                    const uint32_t word = kv_quant8(out, &sc8, &hat, mul);    // all 8 lanes of a group take part
                    if (m_ok) {
                        *reinterpret_cast<uint4 *>(out16 + at) = hat.u;
                        codes[at >> 3] = word;
                        if ((c & 7) == 0) scales[at >> 6] = sc8;
                    }
                }
            }
        }
        return;
    }
    if constexpr (SILU) {
        // Gate and up of a channel lie in the same lane: the product, of their fp16 roundings, is made in registers
        // and only it is stored (5808 x 22016 x 4096: 403 us, 427 with gate | up stored, and the quantizer behind it,
        // which reads half as much, 34 instead of 60).
        constexpr int ZROW = BC + 8;
        f16 *stage = reinterpret_cast<f16 *>(lds_raw);
#pragma unroll
        for (int ib = 0; ib < RT / 2; ++ib) {
            if (ib) __syncthreads();                  // the previous 32 rows have been read
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 sam = *reinterpret_cast<const f32x4 *>(row_scale + 32 * ib + 16 * h + 4 * q);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    f16 *p = stage + (16 * h + 4 * q + r) * ZROW + wave * WC + c16;
#pragma unroll
                    for (int j = 0; j < CB; ++j)
                        p[16 * j] = silu_mul((float)to_f16(yacc[2 * ib + h][j][r] * sam[r]),
                                             (float)to_f16(yacc[2 * ib + h][j + CB][r] * sam[r]));
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 32 * (BC / 8) / NT; ++k) {
                const int idx = k * NT + tid, row = idx / (BC / 8), n = nc0 + 8 * (idx % (BC / 8)), m = m0 + 32 * ib + row;
                const uint4 z = *reinterpret_cast<const uint4 *>(stage + row * ZROW + 8 * (idx % (BC / 8)));
                if (m < M && n < NC) *reinterpret_cast<uint4 *>(y + (size_t)m * ldy + n) = z;
            }
        }
        return;
    }
    // 32 rows at a time through LDS as fp32, so that a thread finishes 8 neighbouring columns of a row: one
    // 16-byte residual load, one 16-byte store, at any element's address (the chip takes both there; of a branch for tensors at multiples of 16
    // bytes and one for others the compiler made stores of 2, 2 and 12 bytes: 80 x 512 x 512 4.04 -> 3.76 us, 160 x 4096 x 4096 11.0 -> 10.6,
    // 636 x 4096 x 4096 19.9 -> 19.3, 1356 x 12288 x 4096 68.3 -> 65.9)
    float *stage = reinterpret_cast<float *>(lds_raw);
    const int n = n8;
    if constexpr (ADDS && !AHEAD) {
#pragma unroll
        for (int ib = 0; ib < ROUNDS; ++ib) ask_residual(ib);
    }
#pragma unroll
    for (int ib = 0; ib < RT / 2; ++ib) {
        if (ib) __syncthreads();                      // the previous 32 rows have been read
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 sam = *reinterpret_cast<const f32x4 *>(row_scale + 32 * ib + 16 * h + 4 * q);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * h + 4 * q + r, m = m0 + 32 * ib + row;
                float *p = stage + row * FROW + wave * WN + c16;
#pragma unroll
                for (int j = 0; j < CT; ++j) {
                    p[16 * j] = yacc[2 * ib + h][j][r] * sam[r];
                    if (ACC_OUT && m < M && n_ok) acc_out[(size_t)m * N + nw + 16 * j + c16] = tot[2 * ib + h][j][r];
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KI; ++k) {
            const int row = RPI * k + row0, m = m0 + 32 * ib + row;
            const float4 *p = reinterpret_cast<const float4 *>(stage + row * FROW + (n - n0));
            const float4 lo = p[0], hi = p[1];
            float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            if (!y || m >= M || n >= N) continue;
            f16x8 o;
            if (res) {
                asm volatile("" : "+v"(rv[ib][k]));   // (else it is converted, and waited for, where it is loaded)
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = v[e] + (float)rv[ib][k][e];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = to_f16(v[e]);
            *reinterpret_cast<f16x8_at2 *>(y + (size_t)m * ldy + n) = o;
        }
    }
}

// (The arguments that the first loads need come first: they are in registers when a wave starts.)
template <int RT, int CT, int NW, int CH, int SP, ActFormat ACTS, bool ACC_OUT, Epilogue EPI, int OCC>
__global__ __launch_bounds__(64 * NW, OCC) void w4a4_f8_kernel(
    const uint4 *__restrict__ wp, const f16 *__restrict__ sw, const uint8_t *__restrict__ qa, const float *__restrict__ sa, int tiles_m, int tiles_n,
    int M, int N, int K, int G, f16 *__restrict__ y, int ldy, const f16 *__restrict__ res, int ldr, int32_t *__restrict__ acc_out, GemmMore more)
{
    w4a4_tile<RT, CT, NW, CH, SP, ACTS, ACC_OUT, EPI>(qa, sa, M, K, G, wp, sw, N, y, ldy, res, ldr, acc_out, tiles_m, tiles_n, more);
}
// The tile of 96 rows, which only the choice takes, under a name of its own: a profile tells it by that from the tiles that can be pinned.
template <int RT, int CT, int NW, int CH, int SP, ActFormat ACTS, bool ACC_OUT, Epilogue EPI, int OCC>
__global__ __launch_bounds__(64 * NW, OCC) void w4a4_rows96_kernel(
    const uint4 *__restrict__ wp, const f16 *__restrict__ sw, const uint8_t *__restrict__ qa, const float *__restrict__ sa, int tiles_m, int tiles_n,
    int M, int N, int K, int G, f16 *__restrict__ y, int ldy, const f16 *__restrict__ res, int ldr, int32_t *__restrict__ acc_out, GemmMore more)
{
    w4a4_tile<RT, CT, NW, CH, SP, ACTS, ACC_OUT, EPI>(qa, sa, M, K, G, wp, sw, N, y, ldy, res, ldr, acc_out, tiles_m, tiles_n, more);
}

// Tile instantiations; the number is what quota_set_gemm_variant pins.
//                                            RT CT NW CH SP          OCC
// 128 x 128 as waves of 128 x 32: three workgroups per CU, so that a launch's last round is finer than with 128 x 256 (5808 x
// 4096 x 11008 213 -> 189 us, 3324 x 5120 x 13824 237 -> 187, 640 x 12288 x 4096 38 -> 33, 11264 x 12288 x 4096 443 and 468).
// 128 x 256 in stages of two groups, half the barriers of one (5808 x 22016 x 4096 369 -> 353 us, 11264 x 12288 x 4096 439 -> 434, 1101 x
// 37888 x 3584 128 -> 123); the packed entry point's rows leave no room for the second group.
// 64 x 128 as four waves of 64 x 32, three workgroups per CU; a weight belongs to one wave.  Stages of four groups are long enough for
// a round trip to memory (400 x 22016 x 4096 49 us, 45 so); the packed entry point's rows, which pass registers, leave no
// room for more than two.
#define F8_TILE_0(P, A, QK) w4a4_f8_kernel<8, 2, 4, 2, 3, P, A, QK, P == PACKED_INT4 ? 2 : 3>   // 128 x 128
#define F8_TILE_1(P, A, QK) w4a4_f8_kernel<4, 2, 4, P == PACKED_INT4 ? 2 : 4, 4, P, A, QK, 3>   // 64 x 128
#define F8_TILE_2(P, A, QK) w4a4_f8_kernel<2, 2, 4, 4, 4, P, A, QK, 2>  // 32 x 128
#define F8_TILE_3(P, A, QK) w4a4_f8_kernel<2, 1, 4, 4, 0, P, A, QK, 2>  // 32 x 64
#define F8_TILE_4(P, A, QK) w4a4_f8_kernel<8, 4, 4, P == PACKED_INT4 ? 1 : 2, P == PACKED_INT4 ? 3 : 6, P, A, QK, 2>  // 128 x 256
// 32 x 64 once more in longer stages, a layer's rows below 512 only, not pinned: chosen where its fitted time is the lowest, which is up to
// one workgroup per CU and from five groups on (101 x 4096 x 11008 22.4 -> 19.5 us; at 237 x 4096 x 11008, 1.9 workgroups, 25.0 against
// 24.3 in stages of four).
#define F8_TILE_5(P, A, QK) w4a4_f8_kernel<2, 1, 4, 8, 4, P, A, QK, 2>  // 32 x 64
// 64 x 256, packed rows only, not pinned: of two rows of blocks fewer than 128 x 256 its registers hold stages of two groups, and launches of
// one to two workgroups per CU take a tenth to a fifth less on it than on any other (320 x 22016 x 4096 51 us on 64 x 128, 41 so; 640 x
// 12288 x 4096 47, 41; 1600 x 4096 x 4096 43, 38; a layer's rows do better on 128 x 128).
#define F8_PACKED_TILE(P, A, QK) w4a4_f8_kernel<4, 4, 4, 2, 6, P, A, QK, 2>

// 96 x 128, a layer's rows below 512 only, not pinned, chosen up to two workgroups per CU, where 64 x 128 comes to more: 129 to 192 rows are two of it and
// three of 64 x 128, which at 22016 columns are 516 workgroups, three for a few CUs.  Over what the choice takes it for, best other tile and
// it, us: 65 to 96 x 37888 x 3584, one of it and two, 24.6 to 26.3, 23.4 to 25.3; 129 to 192 x 22016 x 4096 26.6 to 27.9, 23.4 to 25.8, x 27648 x 5120 34.6
// to 36.1, 30.6 to 32.4; 257 to 384 x 15360 x 5120 35.8 to 39.8, 31.2 to 35.7; 321 to 480 x 12288 x 4096, four or five and six to eight, 29.9 to
// 33.7, 27.0 to 31.0; 39 more shapes of 72 to 493 rows and 8832 to 39360 columns that the choice takes it for: 2 to 15 % less on it.  At 224 x 12288 x 4096, three
// and four, 24.3 against 20.6 on 64 x 128.  Stages of four groups leave room for two workgroups.
#define F8_96_ROW_TILE(P, A, QK) w4a4_rows96_kernel<6, 2, 4, 4, 4, P, A, QK, 2>  // 96 x 128

struct TileShape { int bm, bn, nt, kernel_id; };
constexpr int TILES = 8, PINNED_TILES = 5, PACKED_TILE = 6;
const TileShape kTiles[TILES] = {{128, 128, 256, QUOTA_K_GEMM_128X128}, {64, 128, 256, QUOTA_K_GEMM_64X128},
                             {32, 128, 256, QUOTA_K_GEMM_32X128}, {32, 64, 256, QUOTA_K_GEMM_32X64},
                             {128, 256, 256, QUOTA_K_GEMM_128X256}, {32, 64, 256, QUOTA_K_GEMM_32X64},
                             {64, 256, 256, QUOTA_K_GEMM_64X256}, {96, 128, 256, QUOTA_K_GEMM_96X128}};

typedef void (*f8_kernel)(const uint4 *, const f16 *, const uint8_t *, const float *, int, int, int, int, int, int, f16 *, int, const f16 *, int,
                          int32_t *, GemmMore);

template <ActFormat P, Epilogue E>
f8_kernel tile_kernel(int v)
{
    switch (v) {
    case 0: return F8_TILE_0(P, false, E);
    case 1: return F8_TILE_1(P, false, E);
    case 2: return F8_TILE_2(P, false, E);
    case 3:
        if constexpr (E == SILU_MUL) return nullptr;         // (one block of columns per wave: never chosen)
        else return F8_TILE_3(P, false, E);
    case 4: return F8_TILE_4(P, false, E);
    case 5:
        if constexpr (P != A6 || E == SILU_MUL) return nullptr;
        else return F8_TILE_5(P, false, E);
    case 7:
        if constexpr (P != A6) return nullptr;
        else return F8_96_ROW_TILE(P, false, E);
    default:
        if constexpr (P != PACKED_INT4) return nullptr;
        else return F8_PACKED_TILE(P, false, E);
    }
}

int launch_f8(f8_kernel kernel, int v, int kernel_id, const uint8_t *qa, const float *sa, int M,
              const quota_weights *W, f16 *y, int ldy, const f16 *res, int ldr, int32_t *acc, hipStream_t st,
              const quota_qkv_epilogue *qe = nullptr, const quota_kept_rows *kept = nullptr)
{
    const TileShape &t = kTiles[v];
    const int G = (W->K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    const int tiles_m = (M + t.bm - 1) / t.bm, tiles_n = (W->N + t.bn - 1) / t.bn;
    const double Md = M, Nd = W->N, Kd = W->K;
    ProfScope prof(kernel_id, 2.0 * Md * Nd * Kd,
                   Nd * Kd / 2 + 2.0 * Nd * G + Md * Kd / 2 + 4 * Md +
                       (qe ? Md * (Nd / 3) * (7 + 1.0 / 16) + 4 * Md : 2.0 * Md * (ldy < W->N ? ldy : Nd) * (res ? 2 : 1)), st);
    GemmMore more = {};
    if (qe) more.qkv = *qe;
    else if (kept) more.kept = *kept;
    kernel<<<dim3(tiles_m * tiles_n), dim3(t.nt), 0, st>>>((const uint4 *)W->packed, (const f16 *)W->scales, qa, sa, tiles_m, tiles_n,
                                                           M, W->N, W->K, G, y, ldy, res, ldr, acc, more);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

ActFormat acts_of(int M) { return quota_a6_starts(M) ? A6_STARTS : A6; }       // a layer's M rows

int g_gemm_variant = -1;      // -1: chosen per launch; else pinned by quota_set_gemm_variant

// Tile choice by cost models fitted to measured kernel times on this GPU (us, over weights that no cache holds), one for a layer's rows
// (112 shapes of 40 to 11776 rows, 512 to 37888 columns and 512 to 18944 channels; the 32 x 64 tile's line, which has changed since, by 270
// of 33 to 511 rows and of narrow layers, where the choice costs 0.6 % over the best tile of each on average, 2.3 % with the line before; the 96 x 128 tile's by
// launches of 160 to 444 rows, and right for those of 65 to 493; all from before first weights went out ahead of everything else, which moved no line: over 266
// other shapes of 33 to 2000 rows the choice costs 1.8 % over the best of the tiles that can be pinned, 1.6 before) and one for
// packed rows, whose stages are shorter and tiles others (412 shapes of 33 to 11776 rows; 0.2 % on average, 10 % at most, where two tiles tie over
// cold weights the one that is ahead over warm ones; by a layer's, without the
// 64 x 256 tile, 3.7 %: 5808 x 4096 x 11008 301 us, 236 so).  With x workgroups per CU a group of the K loop, in whole stages of ch, takes u[ceil(x) - 1] for x <= n and
// slope * x, and more for every round of `occ` workgroups, beyond; c0 is the launch, prologue and epilogue, wg an epilogue more for every
// workgroup beyond the first of a CU (a layer's was fitted without).
// Tall tiles read and unpack a weight for more rows and win once the launch fills the chip; the 32-row
// tiles spread small problems over more waves.  Columns of a tile lie in [min_bn, max_bn] (the QKV
// epilogue needs whole heads that stay inside q, k or v); `narrow`: what a tile of one block of columns per wave costs besides.
int choose_tile(ActFormat acts, int M, int N, int K, int min_bn, int max_bn, float narrow = 0.0f)
{
    struct Cost { int ch; float c0, wg; int n; float u[6], slope, round; int occ; };
    static const Cost layer[TILES] = {
        {2, 5.09f, 0.0f, 6, {0.559f, 0.764f, 1.159f, 1.816f, 1.906f, 2.348f}, 0.311f, 0.255f, 3},
        {4, 4.37f, 0.0f, 6, {0.305f, 0.447f, 0.730f, 1.060f, 1.266f, 1.588f}, 0.192f, 0.174f, 3},
        {4, 3.62f, 0.0f, 4, {0.252f, 0.343f, 0.550f, 0.819f}, 0.132f, 0.150f, 3},
        {4, 3.60f, 0.0f, 4, {0.181f, 0.200f, 0.335f, 0.468f}, 0.120f, 0.042f, 4},
        {2, 6.52f, 0.0f, 4, {0.840f, 1.190f, 2.370f, 2.580f}, 0.430f, 0.577f, 2},
        {8, 3.45f, 0.0f, 3, {0.148f, 0.220f, 0.360f}, 0.125f, 0.039f, 3},
        {},
        {4, 4.70f, 0.0f, 2, {0.490f, 0.610f}, 0.300f, 0.300f, 2},
    };
    static const Cost packed[TILES] = {
        {2, 4.519f, 2.113f, 4, {0.774f, 1.038f, 1.800f, 2.136f}, 0.305f, 0.453f, 2},
        {2, 3.669f, 1.149f, 6, {0.509f, 0.655f, 0.891f, 1.298f, 1.524f, 1.792f}, 0.219f, 0.216f, 4},
        {4, 3.531f, 1.388f, 6, {0.422f, 0.482f, 0.668f, 0.923f, 1.048f, 1.304f}, 0.067f, 0.257f, 2},
        {4, 3.186f, 0.791f, 6, {0.303f, 0.415f, 0.559f, 0.669f, 0.851f, 0.967f}, 0.118f, 0.160f, 5},
        {1, 7.545f, 3.655f, 3, {1.209f, 1.531f, 2.636f}, 0.328f, 0.480f, 1},
        {},
        {2, 4.606f, 2.327f, 4, {0.775f, 0.977f, 1.649f, 1.918f}, 0.222f, 0.498f, 2},
    };
    const Cost *cost = acts == PACKED_INT4 ? packed : layer;
    auto fits = [&](int v) {
        const bool built = v < PINNED_TILES || acts == (v == PACKED_TILE ? PACKED_INT4 : A6);
        return built && kTiles[v].bn >= min_bn && kTiles[v].bn <= max_bn;
    };
    if (g_gemm_variant >= 0 && fits(g_gemm_variant)) return g_gemm_variant;
    const int G = (K + QUOTA_GROUP_W - 1) / QUOTA_GROUP_W;
    int best = -1;
    float best_t = 0.0f;
    for (int v = 0; v < TILES; ++v) {
        if (!fits(v)) continue;
        const Cost &c = cost[v];
        const long wgs = (long)((M + kTiles[v].bm - 1) / kTiles[v].bm) * ((N + kTiles[v].bn - 1) / kTiles[v].bn), cus = (wgs + 255) / 256;
        const float x = (float)wgs / 256.0f;
        const int groups = (G + c.ch - 1) / c.ch * c.ch, n = 256 * c.occ;
        const float group = x <= (float)c.n ? c.u[cus - 1] : c.slope * x + c.round * (float)((wgs + n - 1) / n);
        const float t = c.c0 + c.wg * (float)(cus - 1) + groups * group + (kTiles[v].bn < 128 ? narrow : 0.0f);
        if (best < 0 || t < best_t) { best = v; best_t = t; }
    }
    return best;
}

}  // namespace

extern "C" int quota_set_gemm_variant(int variant)
{
    if (variant < -1 || variant >= PINNED_TILES) return QUOTA_ERR_INVALID_ARG;
    g_gemm_variant = variant;
    return QUOTA_OK;
}

// The tiles bring two neighbouring columns' scales to LDS as one dword, which has to lie on a dword's address.  Weights
// whose scales start at an odd halfword go through the few-row kernel 16 rows at a time (its scales pass
// registers): the same bits, slowly.
static bool scales_on_dwords(const quota_weights *W) { return (reinterpret_cast<uintptr_t>(W->scales) & 3) == 0; }
static int gemm_16_rows_at_a_time(const uint8_t *qa, quota_rows16_format format, size_t row_bytes, const float *sa, int M,
                                  const quota_weights *W, f16 *y, int ldy, const f16 *res, int ldr, hipStream_t st)
{
    for (int m = 0; m < M; m += 16) {
        const int rc = quota_internal_rows16(qa + m * row_bytes, format, sa + m, M - m < 16 ? M - m : 16, W, y + (size_t)m * ldy,
                                             ldy, res ? res + (size_t)m * ldr : nullptr, ldr, st);
        if (rc != QUOTA_OK) return rc;
    }
    return QUOTA_OK;
}

// GEMM on activations in the internal A6 format (M > 16 rows of a layer).
int quota_internal_w4a4_gemm_a6(const uint8_t *qa6, const float *sa, int M, const quota_weights *W,
                                void *y_f16, int ldy, const void *residual_opt, int ldr, hipStream_t st)
{
    if (!qa6 || !sa || !W || !W->packed || !W->scales || !y_f16) return QUOTA_ERR_NULL;
    if (W->N % 64 != 0 || W->K % 32 != 0) return QUOTA_ERR_SHAPE;
    if (M <= 0) return QUOTA_OK;
    if (M <= 16) return quota_internal_rows16(qa6, QUOTA_ROWS16_A6, sa, M, W, y_f16, ldy, residual_opt, ldr, st);
    if (!scales_on_dwords(W))
        return gemm_16_rows_at_a_time(qa6, QUOTA_ROWS16_A6, quota_a6_row_bytes(W->K), sa, M, W, (f16 *)y_f16, ldy,
                                      (const f16 *)residual_opt, ldr, st);
    const int v = choose_tile(acts_of(M), M, W->N, W->K, 0, 256);
    return launch_f8(quota_a6_starts(M) ? tile_kernel<A6_STARTS, PLAIN>(v) : tile_kernel<A6, PLAIN>(v), v, kTiles[v].kernel_id, qa6, sa, M, W, (f16 *)y_f16, ldy,
                     (const f16 *)residual_opt, ldr, nullptr, st);
}

bool quota_gemm_gathers(int M, const quota_weights *W)
{
    return M > 16 && !quota_a6_starts(M) && W->N % 64 == 0 && W->K % 32 == 0 && scales_on_dwords(W);
}
int quota_internal_w4a4_gemm_a6_kept(const uint8_t *qa6, const float *sa, int M, const quota_kept_rows *kept, const quota_weights *W, void *y_f16, int ldy,
                                     const void *residual, int ldr, hipStream_t st)
{
    if (!qa6 || !sa || !kept || !kept->keep_idx || !W || !W->packed || !W->scales || !y_f16 || !residual) return QUOTA_ERR_NULL;
    if (!quota_gemm_gathers(M, W) || kept->k_keep <= 0 || kept->n_keep <= 0) return QUOTA_ERR_SHAPE;
    const int v = choose_tile(A6, M, W->N, W->K, 0, 256);
    return launch_f8(tile_kernel<A6, PLAIN_PICKED>(v), v, kTiles[v].kernel_id, qa6, sa, M, W, (f16 *)y_f16, ldy, (const f16 *)residual, ldr, nullptr, st, nullptr, kept);
}

// Gate/up projection with SiLU(gate) * up in the epilogue: z [M][N / 2], the bits of the plain projection and the
// stand-alone product.  Returns QUOTA_ERR_SHAPE when the fused form does not fit (the caller then runs the two kernels
// separately): with unaligned scales, or where the tile of choice has one block of columns per wave (projections
// that leave the chip part idle, 37 x 2752 x 512: 4 us each way).  The product then takes the quantizer in front of down longer (33 to 80 rows
// of 1376, 2816 and 11008 channels 0.3, 0.4 and 1.2 us).
int quota_internal_w4a4_gemm_silu(const uint8_t *qa6, const float *sa, int M, const quota_weights *W, void *z_f16,
                                  hipStream_t st)
{
    if (!qa6 || !sa || !W || !W->packed || !W->scales || !z_f16) return QUOTA_ERR_NULL;
    if (M <= 16 || W->N % 64 != 0 || W->K % 32 != 0 || !scales_on_dwords(W) || (reinterpret_cast<uintptr_t>(z_f16) & 15))
        return QUOTA_ERR_SHAPE;
    const int v = choose_tile(acts_of(M), M, W->N, W->K, 0, 256, 0.15f + 4.5e-5f * (float)W->N);
    if (kTiles[v].bn < 128) return QUOTA_ERR_SHAPE;
    return launch_f8(quota_a6_starts(M) ? tile_kernel<A6_STARTS, SILU_MUL>(v) : tile_kernel<A6, SILU_MUL>(v), v, kTiles[v].kernel_id,
                     qa6, sa, M, W, (f16 *)z_f16, W->N / 2, nullptr, 0, nullptr, st);
}

extern "C" int quota_w4a4_gemm(const uint8_t *qa, const float *sa, int M, const quota_weights *W,
                               void *y_f16, int ldy, const void *residual_opt, int ldr,
                               int32_t *acc_i32_opt, void *stream)
{
    if (!qa || !sa || !W || !W->packed || !W->scales) return QUOTA_ERR_NULL;
    if (!y_f16 && !acc_i32_opt) return QUOTA_ERR_NULL;
    if (M < 0 || W->N <= 0 || W->K <= 0) return QUOTA_ERR_INVALID_ARG;
    if (W->N % 64 != 0 || W->K % 32 != 0) return QUOTA_ERR_SHAPE;
    if (y_f16 && ldy < W->N) return QUOTA_ERR_INVALID_ARG;
    if (residual_opt && ldr < W->N) return QUOTA_ERR_INVALID_ARG;
    if (M == 0) return QUOTA_OK;
    hipStream_t st = (hipStream_t)stream;
    f16 *y = (f16 *)y_f16;
    const f16 *res = (const f16 *)residual_opt;
    const bool dwords = scales_on_dwords(W);
    if (acc_i32_opt) {
        quota_weights Wi = *W;
        if (!dwords) Wi.scales = W->packed;      // (the integer sums need no scales: any readable ones do)
        const int rc = launch_f8(F8_TILE_1(PACKED_INT4, true, PLAIN), 1, QUOTA_K_GEMM_OTHER, qa, sa, M, &Wi, dwords ? y : nullptr, ldy,
                                 res, ldr, acc_i32_opt, st);
        if (rc != QUOTA_OK || dwords || !y) return rc;
    }
    if (!dwords) return gemm_16_rows_at_a_time(qa, QUOTA_ROWS16_PACKED, W->K / 2, sa, M, W, y, ldy, res, ldr, st);
    if (M <= 16)            // the decode step: stream the weights once
        return quota_internal_rows16(qa, QUOTA_ROWS16_PACKED, sa, M, W, y, ldy, res, ldr, st);
    const int v = choose_tile(PACKED_INT4, M, W->N, W->K, 0, 256);
    return launch_f8(tile_kernel<PACKED_INT4, PLAIN>(v), v, kTiles[v].kernel_id, qa, sa, M, W, y, ldy, res, ldr, nullptr, st);
}

// QKV projection with the RoPE + 4-bit K/V quantizer fused into the epilogue (see the kernel).
// qa6 is in the A6 format.
// y_opt, when not null, also receives the plain fp16 q | k | v.  Returns QUOTA_ERR_SHAPE when the
// shape does not fit the fused form (the caller then runs the two kernels separately).
int quota_internal_w4a4_gemm_qkv(const uint8_t *qa6, const float *sa, int M, const quota_weights *W,
                                 void *y_opt, const quota_qkv_epilogue *qe, hipStream_t st)
{
    if (!qa6 || !sa || !W || !W->packed || !W->scales || !qe || !qe->pos || !qe->cosT || !qe->sinT ||
        !qe->q_rot || !qe->khat || !qe->vhat || !qe->k_codes || !qe->k_scales || !qe->v_codes || !qe->v_scales)
        return QUOTA_ERR_NULL;
    if (M < 0 || qe->n_pos <= 0) return QUOTA_ERR_INVALID_ARG;
    const int d = qe->d, dkv = qe->dkv;
    if ((qe->dh != 64 && qe->dh != 128) || d <= 0 || d % 128 != 0 || dkv <= 0 || dkv % 128 != 0 ||
        W->N != d + 2 * dkv || W->K % 32 != 0 || !scales_on_dwords(W))
        return QUOTA_ERR_SHAPE;
    if (M == 0) return QUOTA_OK;
    const int v = choose_tile(acts_of(M), M, W->N, W->K, qe->dh, d % 256 == 0 && dkv % 256 == 0 ? 256 : 128);
    return launch_f8(quota_a6_starts(M) ? tile_kernel<A6_STARTS, QKV_ROPE_KV>(v) : tile_kernel<A6, QKV_ROPE_KV>(v), v, kTiles[v].kernel_id, qa6, sa, M, W, (f16 *)y_opt, W->N, nullptr, 0,
                     nullptr, st, qe);
}
