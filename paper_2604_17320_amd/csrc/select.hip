// Token scoring (Eq. 6-8) and deterministic budgeted top-k (Eq. 9).
// One workgroup per sequence: a chain of small steps, bound by their latencies.  Order statistics and the top-k
// threshold come from an exact radix select on order-preserving uint32 keys, 8 bits a pass from the highest bit
// in which any two keys differ (a float key's top byte is nearly constant: taken as the first digit, all lanes of
// a wave add to the same few counters, one after the other); the counters are integers, so the result does not depend
// on execution order.  Up to 1024 tokens each select is one wave's, without a barrier (small_score_topk_kernel).  Beyond, all
// waves take part, with their keys in registers: four per metric, both percentile bounds in the same passes, then all
// sixteen for the top-k; a select ends as soon as at most 64 keys share a rank's digits, which one wave ranks (2880 tokens
// 18.8 us; one wave per bound and per top-k with the head means of the attention cues took 113).
#include "common.h"
#include "internal.h"
#include <type_traits>
#include "prefetch.h"
#include "headmeans.h"
#include "rowquant.h"

namespace {

constexpr int MAXV = QUOTA_MAX_SCORED_TOKENS;

// ascending uint32 order == ascending float order; -0 is folded onto +0
__device__ __forceinline__ uint32_t float_key(float f)
{
    f = f + 0.0f;
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k)
{
    uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves (no LDS crossbar): shifts by
// 1, 2, 4, 8 inside each row of 16 lanes, then lane 15 of rows 0 and 2 is added to rows 1 and 3,
// then lane 31 to rows 2 and 3.  Lanes without a source add 0.
__device__ __forceinline__ int wave_incl_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);     // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);     // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);     // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);     // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15 -> rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31 -> rows 2, 3
    return v;
}

__device__ __forceinline__ uint32_t wave_umax(uint32_t v)
{
#define STEP(ctrl, rows) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, rows, 0xf, false));
    QUOTA_DPP_STEPS(STEP)
#undef STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

constexpr int SCORE_THREADS = 1024, SCORE_WAVES = SCORE_THREADS / 64, SELECT_RANGE = 2 * SCORE_WAVES + 32;

// Exact rank[r]-th smallest (0-based) of the n keys of a group of GT threads (key j of thread t of the group is number
// t + GT j), for NR ranks at once; all SCORE_THREADS threads call this, SCORE_THREADS / GT groups work side by
// side.  hist: 3 NR 256 ints of LDS per group (a pass clears the next one's counters), range: SELECT_RANGE
// words of LDS.  Every thread of the group gets its results.
template <int GT, int PERG, int NR>
__device__ void group_select(const uint32_t (&key)[PERG], int n, const int (&rank)[NR], uint32_t (&result)[NR],
                             int *hist, uint32_t *range)
{
    const int tid = threadIdx.x, lane = tid & 63, gt = tid % GT;
    constexpr int WPG = GT / 64;                    // waves per group
    uint32_t kmax = 0, kinv = 0;                    // largest key, largest complement of a key
#pragma unroll
    for (int j = 0; j < PERG; ++j)
        if (gt + GT * j < n) {
            kmax = max(kmax, key[j]);
            kinv = max(kinv, ~key[j]);
        }
    kmax = wave_umax(kmax);
    kinv = wave_umax(kinv);
    if (lane == 0) {
        range[2 * (tid >> 6)] = kmax;
        range[2 * (tid >> 6) + 1] = kinv;
    }
    for (int i = gt; i < NR * 256; i += GT) hist[i] = 0;
    __syncthreads();
    int bits = 0, most = 0;                         // low bits in which this group's / any group's keys differ
    uint32_t kmin = 0;
#pragma unroll
    for (int g = 0; g < SCORE_WAVES / WPG; ++g) {
        uint32_t hi = 0, lo = 0;
#pragma unroll
        for (int w = 0; w < WPG; ++w) {
            hi = max(hi, range[2 * (g * WPG + w)]);
            lo = max(lo, range[2 * (g * WPG + w) + 1]);
        }
        const int differ = hi == ~lo ? 0 : 32 - __clz((int)(hi ^ ~lo));
        most = max(most, differ);
        if (g == tid / GT) { bits = differ; kmin = ~lo; }
    }
    uint32_t mask = bits == 32 ? 0u : ~0u << bits, prefix[NR];
    int remaining[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) { prefix[r] = kmin & mask; remaining[r] = rank[r]; }
    // per rank of every group: digit and rank among its keys, whether those are too many for a wave, the result
    int *found = reinterpret_cast<int *>(range) + 2 * SCORE_WAVES + 2 * NR * (tid / GT);
    int *many = reinterpret_cast<int *>(range) + 2 * SCORE_WAVES + 16;
    uint32_t *chosen = range + 2 * SCORE_WAVES + 24 + NR * (tid / GT);
    constexpr int RANKS = NR * SCORE_WAVES / WPG;
    bool few = false;
    int *list = hist;                                // the counters cleared last
    for (int pass = 0, at = 0; 8 * pass < most && !few; ++pass) {
        const int next = at == 2 ? 0 : at + 1, width = min(8, bits), shift = bits - width;
        int *h = hist + at * NR * 256, *hn = hist + next * NR * 256;
        const uint32_t digits = (1u << width) - 1;
        const bool split = NR > 1 && prefix[NR - 1] != prefix[0];
        if (width > 0) {
#pragma unroll
            for (int j = 0; j < PERG; ++j) {
                if (gt + GT * j >= n) continue;
                if ((key[j] & mask) == prefix[0]) atomicAdd(&h[(key[j] >> shift) & digits], 1);
                if (split && (key[j] & mask) == prefix[NR - 1]) atomicAdd(&h[256 + ((key[j] >> shift) & digits)], 1);
            }
        }
        for (int i = gt; i < NR * 256; i += GT) hn[i] = 0;
        __syncthreads();
        // one wave per rank finds the digit (spread over the SIMDs)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if ((tid >> 6) % WPG != (NR * (tid / GT) + r) % WPG) continue;
            if (width == 0) {                       // (all bits known: the key is the prefix)
                if (lane == 0) many[NR * (tid / GT) + r] = 0;
                continue;
            }
            const i32x4 c = *reinterpret_cast<const i32x4 *>(h + (split ? 256 * r : 0) + 4 * lane);
            const int sum = c[0] + c[1] + c[2] + c[3], incl = wave_incl_scan(sum), excl = incl - sum;
            int left = remaining[r] - excl, digit = 4 * lane, keys = c[0];
            const bool mine = left >= 0 && remaining[r] < incl;         // exactly one lane
            if (left >= c[0]) { left -= c[0]; ++digit; keys = c[1];
                if (left >= c[1]) { left -= c[1]; ++digit; keys = c[2];
                    if (left >= c[2]) { left -= c[2]; ++digit; keys = c[3]; } } }
            if (mine) {
                found[2 * r] = digit;
                found[2 * r + 1] = left;
                many[NR * (tid / GT) + r] = keys > 64 && shift > 0;
            }
        }
        __syncthreads();
        if (width > 0) {
            mask |= digits << shift;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                prefix[r] |= (uint32_t)found[2 * r] << shift;
                remaining[r] = found[2 * r + 1];
            }
            bits = shift;
        }
        few = true;
#pragma unroll
        for (int i = 0; i < RANKS; ++i) few = few && !many[i];
        list = hn;
        at = next;
    }
    // At most 64 keys share a rank's digits, mostly after one or two of four passes: a wave ranks them among each other
    if (few) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (bits == 0) {
                if (gt == 0) chosen[r] = prefix[r];
                continue;
            }
#pragma unroll
            for (int j = 0; j < PERG; ++j)
                if (gt + GT * j < n && (key[j] & mask) == prefix[r])
                    list[256 * r + atomicAdd(&list[256 * r + 255], 1)] = (int)key[j];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (bits == 0 || (tid >> 6) % WPG != (NR * (tid / GT) + r) % WPG) continue;
            const int keys = __builtin_amdgcn_readfirstlane(list[256 * r + 255]);
            const uint32_t mine = (uint32_t)list[256 * r + min(lane, keys - 1)];
            int below = 0, upto = 0;
            for (int i = 0; i < keys; ++i) {
                const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
                below += k < mine;
                upto += k <= mine;
            }
            if (below <= remaining[r] && remaining[r] < upto) chosen[r] = mine;      // (lanes of equal keys agree)
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) result[r] = few ? chosen[r] : prefix[r];
}

// G (Eq. 7): clip to the nearest-rank percentiles and rescale to [0, 1]
__device__ __forceinline__ float robust_unit(float m, float lo, float hi)
{
    if (hi == lo) return 0.5f;
    float num = m - lo;
    float den = hi - lo;
    float v = num / den;
    return fminf(fmaxf(v, 0.0f), 1.0f);
}

// Eq. 8, in the order it is written
__device__ __forceinline__ float fuse_score(const quota_score_params &p, float g0, float g1, float g2, float g3)
{
    float a = p.w_m * g0;
    float c = p.w_c * g1;
    float s = p.w_s * g2;
    float rr = p.w_r * g3;
    float acc = a + c;
    acc = acc + s;
    return acc + rr;
}

struct MetricSrc {
    const float *sumsq, *ressq, *cm_inter, *cm_intra;
    size_t osq, ocm;        // offsets of this sequence in the sumsq/ressq and cm arrays
};

// Loads the four Eq. 6 metrics of sequence b into LDS as order-preserving keys, finds the
// eight percentile bounds, then fuses the score of every token; key[r] is the order-preserving key of the score
// of token tid + 1024 r (0 for NaN: ranks lowest).
// mk: 4*cap keys (cap >= Nv: the stride between the four metrics), hist: 4 * 3 * 2 * 256 ints, range: SELECT_RANGE words.
template <int PER>      // tokens per thread of the fusion pass: Nv <= PER * SCORE_THREADS
__device__ void score_phase(const MetricSrc &src, int B, int Nv, int b, const quota_score_params &p,
                            float *__restrict__ score, float *__restrict__ normed, uint32_t *mk, int cap,
                            int *hist, uint32_t *range, float *lohi, uint32_t (&key)[PER])
{
    const int tid = threadIdx.x;
    for (int i = tid; i < Nv; i += SCORE_THREADS) {
        mk[1 * cap + i] = float_key(src.cm_inter[src.ocm + i]);
        mk[2 * cap + i] = float_key(src.cm_intra[src.ocm + i]);
        mk[0 * cap + i] = float_key(sqrtf(src.sumsq[src.osq + i]));    // m_mag
        mk[3 * cap + i] = float_key(sqrtf(src.ressq[src.osq + i]));    // m_res
    }
    __syncthreads();
    const int r_lo = (p.pct_lo * (Nv - 1) + 50) / 100, r_hi = (p.pct_hi * (Nv - 1) + 50) / 100;
    {
        constexpr int GT = SCORE_THREADS / 4;
        const int m = tid / GT, rank[2] = {r_lo, r_hi};
        uint32_t mkey[4 * PER], bound[2];
#pragma unroll
        for (int j = 0; j < 4 * PER; ++j) mkey[j] = mk[m * cap + min(tid % GT + GT * j, Nv - 1)];
        group_select<GT, 4 * PER, 2>(mkey, Nv, rank, bound, hist + m * 3 * 2 * 256, range);
        if (tid % GT == 0) {
            lohi[2 * m] = key_float(bound[0]);
            lohi[2 * m + 1] = key_float(bound[1]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int i = tid + SCORE_THREADS * r;
        if (i < Nv) {
            float g0 = robust_unit(key_float(mk[0 * cap + i]), lohi[0], lohi[1]);
            float g1 = robust_unit(key_float(mk[1 * cap + i]), lohi[2], lohi[3]);
            float g2 = robust_unit(key_float(mk[2 * cap + i]), lohi[4], lohi[5]);
            float g3 = robust_unit(key_float(mk[3 * cap + i]), lohi[6], lohi[7]);
            const float acc = fuse_score(p, g0, g1, g2, g3);
            size_t o = (size_t)b * Nv + i;
            score[o] = acc;
            key[r] = acc != acc ? 0u : float_key(acc);
            if (normed) {
                size_t plane = (size_t)B * Nv;
                normed[0 * plane + o] = g0;
                normed[1 * plane + o] = g1;
                normed[2 * plane + o] = g2;
                normed[3 * plane + o] = g3;
            }
        }
    }
}

// Indices of the K largest of the Nv keys (key r of thread t is number t + 1024 r), ties to the lower index, ascending.
// Requires 0 < K < Nv.  counts: 2 * PER * SCORE_WAVES ints of LDS.
template <int PER>
__device__ void topk_phase(const uint32_t (&key)[PER], int Nv, int K, int32_t *__restrict__ out, int *hist,
                           uint32_t *range, int *counts)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // threshold = K-th largest = rank (Nv - K) in ascending order
    const int rank[1] = {Nv - K};
    uint32_t thr[1];
    group_select<SCORE_THREADS, PER, 1>(key, Nv, rank, thr, hist, range);
    // 64 consecutive tokens per wave and r: how many are above / at the threshold
    unsigned long long gt[PER], eq[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const bool live = tid + SCORE_THREADS * r < Nv;
        gt[r] = __ballot(live && key[r] > thr[0]);
        eq[r] = __ballot(live && key[r] == thr[0]);
        if (lane == 0) {
            counts[2 * (r * SCORE_WAVES + wave)] = __popcll(gt[r]);
            counts[2 * (r * SCORE_WAVES + wave) + 1] = __popcll(eq[r]);
        }
    }
    __syncthreads();
    // counts before each run of 64, by every wave for itself: lane l holds runs 2 l, 2 l + 1
    constexpr int RUNS = PER * SCORE_WAVES;
    int g0 = 0, g1 = 0, e0 = 0, e1 = 0;
    if (2 * lane < RUNS) { g0 = counts[4 * lane]; e0 = counts[4 * lane + 1]; g1 = counts[4 * lane + 2]; e1 = counts[4 * lane + 3]; }
    const int gi = wave_incl_scan(g0 + g1), ei = wave_incl_scan(e0 + e1);
    const int need = K - __builtin_amdgcn_readlane(gi, 63);        // ties taken, lowest indices first
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int run = r * SCORE_WAVES + wave, from = run >> 1;
        int gb = __shfl(gi - g0 - g1, from, 64), eb = __shfl(ei - e0 - e1, from, 64);
        if (run & 1) { gb += __shfl(g0, from, 64); eb += __shfl(e0, from, 64); }
        const unsigned long long below = (1ull << lane) - 1;
        gb += __popcll(gt[r] & below);
        eb += __popcll(eq[r] & below);
        const bool above = gt[r] >> lane & 1, at = eq[r] >> lane & 1;
        if (above || (at && eb < need)) out[gb + min(eb, need)] = tid + SCORE_THREADS * r;
    }
}

constexpr int SELECT_HIST = 4 * 3 * 2 * 256;      // counters of four two-rank selects

// K < 0: score only.  When K >= 0 the indices of the min(K, Nv) best tokens of
// sequence b go to keep_idx[b][0..min(K,Nv)).
template <int PER, typename PRE>
__global__ __launch_bounds__(SCORE_THREADS) void score_topk_kernel(MetricSrc src, long stride_sq, int B, int Nv,
                                                         quota_score_params p,
                                                         float *__restrict__ score,
                                                         float *__restrict__ normed, int K,
                                                         int32_t *__restrict__ keep_idx, int cap, PRE pre)
{
    if ((int)blockIdx.x >= B) {
        prefetch<SCORE_THREADS>(pre, blockIdx.x - B, gridDim.x - B);
        return;
    }
    // LDS sized by the launch for this Nv: counters, ranges and bounds, 4 * cap keys
    extern __shared__ __align__(16) uint32_t score_lds[];
    int *hist = reinterpret_cast<int *>(score_lds);
    uint32_t *range = score_lds + SELECT_HIST;
    float *lohi = reinterpret_cast<float *>(range + SELECT_RANGE);
    uint32_t *mk = range + SELECT_RANGE + 8;
    const int b = blockIdx.x;
    src.osq = (size_t)b * stride_sq;
    src.ocm = (size_t)b * Nv;
    uint32_t key[PER];
    score_phase<PER>(src, B, Nv, b, p, score, normed, mk, cap, hist, range, lohi, key);
    if (K < 0) return;
    const int k = K < Nv ? K : Nv;
    int32_t *out = keep_idx + (size_t)b * k;
    if (k == Nv) {
        for (int i = threadIdx.x; i < Nv; i += SCORE_THREADS) out[i] = i;
        return;
    }
    if (k == 0) return;
    __syncthreads();            // the counters and keys have been read
    topk_phase<PER>(key, Nv, k, out, hist, range, (int *)mk);
}

// ---- up to SCORE_THREADS tokens: each select by a wave of its own, whose 64 lanes hold all keys (key i in register i / 64 of lane
// i % 64) and whose counters no other wave touches, so that it needs no barrier: eight waves find the percentile bounds, one the
// top-k.
constexpr int WAVE_KEYS = SCORE_THREADS / 64;

// run(r) for the registers that hold keys, four at a time
template <typename RUN>
__device__ __forceinline__ void for_keys(int n, RUN run)
{
#pragma unroll
    for (int r4 = 0; r4 < WAVE_KEYS; r4 += 4)
        if (64 * r4 < n)
#pragma unroll
            for (int r = r4; r < r4 + 4; ++r) run(r);
}
// load(i): key i
template <typename LOAD>
__device__ __forceinline__ void wave_keys(int n, uint32_t (&key)[WAVE_KEYS], LOAD load)
{
    for_keys(n, [&](int r) { key[r] = load(min(64 * r + (int)(threadIdx.x & 63), n - 1)); });
}
// The rank-th smallest (0-based) of a wave's n keys; h: 256 ints of LDS.
__device__ __forceinline__ uint32_t wave_select(const uint32_t (&key)[WAVE_KEYS], int n, int rank, int *h)
{
    const int lane = threadIdx.x & 63;
    uint32_t kmax = 0, kinv = 0;                     // (past the last key its copies)
    for_keys(n, [&](int r) {
        kmax = max(kmax, key[r]);
        kinv = max(kinv, ~key[r]);
    });
    kmax = wave_umax(kmax);
    const uint32_t kmin = ~wave_umax(kinv);
    if (kmin == kmax) return kmin;
    int bits = 32 - __clz((int)(kmin ^ kmax)), left = rank;
    uint32_t mask = bits == 32 ? 0u : ~0u << bits, prefix = kmin & mask;
    while (true) {
        const int width = min(8, bits), shift = bits - width;
        const uint32_t digits = (1u << width) - 1;
        *reinterpret_cast<i32x4 *>(h + 4 * lane) = i32x4{0, 0, 0, 0};
        __builtin_amdgcn_wave_barrier();             // (a wave's accesses to LDS stay in their order)
        for_keys(n, [&](int r) {
            if ((key[r] & mask) == prefix && 64 * r + lane < n) atomicAdd(&h[(key[r] >> shift) & digits], 1);
        });
        __builtin_amdgcn_wave_barrier();
        const i32x4 c = *reinterpret_cast<const i32x4 *>(h + 4 * lane);
        __builtin_amdgcn_wave_barrier();
        const int incl = wave_incl_scan(c[0] + c[1] + c[2] + c[3]);
        // the first lane whose counters reach past the rank, and the counter there
        const int from = __builtin_ctzll(__ballot(left < incl));
        const int c0 = __builtin_amdgcn_readlane(c[0], from), c1 = __builtin_amdgcn_readlane(c[1], from),
                  c2 = __builtin_amdgcn_readlane(c[2], from), c3 = __builtin_amdgcn_readlane(c[3], from);
        left -= __builtin_amdgcn_readlane(incl, from) - (c0 + c1 + c2 + c3);
        int digit = 4 * from, keys = c0;
        if (left >= c0) { left -= c0; ++digit; keys = c1;
            if (left >= c1) { left -= c1; ++digit; keys = c2;
                if (left >= c2) { left -= c2; ++digit; keys = c3; } } }
        prefix |= (uint32_t)digit << shift;
        mask |= digits << shift;
        bits = shift;
        if (bits == 0) return prefix;
        if (keys == 1) {                             // mostly after one or two of four passes
            uint32_t found = prefix;
            for_keys(n, [&](int r) {
                const unsigned long long in = __ballot((key[r] & mask) == prefix);
                if (in) found = (uint32_t)__builtin_amdgcn_readlane((int)key[r], __builtin_ctzll(in));
            });
            return found;
        }
    }
}

// first + the lanes below this one in a ballot
__device__ __forceinline__ int count_before(unsigned long long ballot, int first)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ballot, first));
}
// One wave: indices of the K largest of the Nv keys, ties to the lower index, ascending; 0 < K < Nv.
__device__ __forceinline__ void wave_topk(const uint32_t (&key)[WAVE_KEYS], int Nv, int K, int32_t *__restrict__ out, int *h)
{
    const int lane = threadIdx.x & 63;
    const uint32_t thr = wave_select(key, Nv, Nv - K, h);       // K-th largest
    int need = K;                                    // ties taken, lowest indices first
    for_keys(Nv, [&](int r) { need -= __popcll(__ballot(key[r] > thr && 64 * r + lane < Nv)); });
    int gb = 0, eb = 0;                              // above, at the threshold so far
    for_keys(Nv, [&](int r) {
        const bool live = 64 * r + lane < Nv, above = live && key[r] > thr, at = live && key[r] == thr;
        const unsigned long long gt = __ballot(above), eq = __ballot(at);
        const int g = count_before(gt, gb), e = count_before(eq, eb);
        if (above || (at && e < need)) out[g + min(e, need)] = 64 * r + lane;
        gb += __popcll(gt);
        eb += __popcll(eq);
    });
}

// score_topk_kernel for up to SCORE_THREADS tokens: one by each thread, beside the eight bounds by a wave each.  Three barriers in
// front of the output and two around the counts in it, where a select by all waves takes three for every pass: 64 / 256 / 576 / 1000 tokens 6.7 /
// 7.6 / 8.7 / 10.0 -> 4.5 / 5.2 / 7.0 / 8.8 us (with the output by the one wave too 576 tokens 7.8).
struct MeansThere {};            // (the cues' head means are in src)
// Workgroups between the sequences' and the fetching ones: four rows each, a quarter of the threads to a row.
struct NoRows {
    __device__ __forceinline__ int wgs() const { return 0; }
    __device__ __forceinline__ void operator()(int) const {}
};
template <int NCH>
struct RowsBeside {
    quota_rows_beside r;
    __host__ __device__ __forceinline__ int wgs() const { return (r.M + 3) / 4; }
    __device__ __forceinline__ void operator()(int wg) const
    {
        __shared__ float top[SCORE_WAVES];
        const int lane = threadIdx.x & 255, quarter = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
        const int row = min(4 * wg + quarter, r.M - 1), nchunk = r.d >> 3;       // (past the last: the same once more)
        const uint4 *xr = reinterpret_cast<const uint4 *>(r.x + (size_t)row * r.d);
        Pack16 v[NCH];
#pragma unroll
        for (int i = 0; i < NCH; ++i) v[i].u = xr[min(lane + 256 * i, nchunk - 1)];
        E6Store store;
        store.make(lane, row);
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < NCH; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf((float)v[i].h[e]));       // (a clamped chunk repeats one of the row's)
        a = wave_absmax(a);
        if ((threadIdx.x & 63) == 0) top[threadIdx.x >> 6] = a;
        __syncthreads();
        a = fmaxf(fmaxf(top[4 * quarter], top[4 * quarter + 1]), fmaxf(top[4 * quarter + 2], top[4 * quarter + 3]));
        float s;
        quantize_cached_row<false, 256, NCH>(v, nchunk, lane, a, row_out(RowOutA6{r.q}, row, nchunk), store, s);
        if (lane == 0) r.scale[row] = s;
    }
};
template <typename MEANS, typename PRE, typename ROWS>
__global__ __launch_bounds__(SCORE_THREADS) void small_score_topk_kernel(const float *sumsq, const float *ressq, const float *cm_inter,
                                                                         const float *cm_intra, int B, int Nv, int K, int stride_sq,
                                                                         float *__restrict__ score, int32_t *__restrict__ keep_idx, float *__restrict__ normed,
                                                                         quota_score_params p, MEANS cues, PRE pre, ROWS rows)
{
    MetricSrc src{sumsq, ressq, cm_inter, cm_intra, 0, 0};       // (plain arguments, the first ones in front: in registers when a wave starts)
    if ((int)blockIdx.x >= B) {
        const int beside = rows.wgs(), wg = blockIdx.x - B;
        if (wg < beside) rows(wg);
        else prefetch<SCORE_THREADS>(pre, wg - beside, gridDim.x - B - beside);
        return;
    }
    __shared__ __align__(16) int counters[8][256];
    __shared__ float lohi[8];
    __shared__ uint32_t scores[SCORE_THREADS], threshold;
    __shared__ int counts[SCORE_WAVES];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), b = blockIdx.x, at = min(tid, Nv - 1);
    src.osq = (size_t)b * stride_sq;
    src.ocm = (size_t)b * Nv;
    constexpr bool TAKES_MEANS = std::is_same<MEANS, quota_cue_masses>::value;
    __shared__ float means[2][TAKES_MEANS ? SCORE_THREADS : 1];
    const float *inter = TAKES_MEANS ? means[0] : src.cm_inter + src.ocm, *intra = TAKES_MEANS ? means[1] : src.cm_intra + src.ocm;
    float m[4] = {src.sumsq[src.osq + at], 0.0f, 0.0f, src.ressq[src.osq + at]};
    // (asked for here, while the metrics are on their way, not between the selects: their first touch comes from far away)
    asm volatile("" ::"s"(score), "s"(keep_idx), "s"(normed));
    if constexpr (TAKES_MEANS) {
        const float invH = 1.0f / (float)cues.H;
        for (int i = tid >> 2; i < Nv; i += SCORE_THREADS / 4) {         // (the lanes of a quad stay together)
            const float2 sums = head_sums(cues.partial + (size_t)b * cues.H * Nv, cues.H, Nv, i, tid & 3);
            if ((tid & 3) == 0) {
                means[0][i] = sums.x * invH;
                means[1][i] = sums.y * invH;
                cues.cm_inter[src.ocm + i] = sums.x * invH;
                cues.cm_intra[src.ocm + i] = sums.y * invH;
            }
        }
        __syncthreads();
    }
    m[1] = inter[at];
    m[2] = intra[at];
    if (wave < 8) {                                  // metric wave / 2, one of its bounds
        const float *from = wave < 2 ? src.sumsq + src.osq : wave < 4 ? inter : wave < 6 ? intra : src.ressq + src.osq;
        // The squares order as their roots do (the root is rounded to nearest, which keeps order), so that only the bound's root is
        // taken; not where a caller hands in a negative number, whose root is none.
        bool roots = wave < 2 || wave >= 6, negative = false;
        uint32_t key[WAVE_KEYS];
        wave_keys(Nv, key, [&](int i) { return __float_as_uint(from[i]); });
        for_keys(Nv, [&](int r) { negative = negative || __uint_as_float(key[r]) < 0.0f; });
        if (roots && __ballot(negative)) {
            roots = false;
            for_keys(Nv, [&](int r) { key[r] = __float_as_uint(sqrtf(__uint_as_float(key[r]))); });
        }
        for_keys(Nv, [&](int r) { key[r] = float_key(__uint_as_float(key[r])); });
        const int pct = wave & 1 ? p.pct_hi : p.pct_lo;
        float bound = key_float(wave_select(key, Nv, (pct * (Nv - 1) + 50) / 100, counters[wave]));
        if (roots) bound = sqrtf(bound);
        if ((tid & 63) == 0) lohi[wave] = bound;
    }
    __syncthreads();
    if (tid < Nv) {
        m[0] = sqrtf(m[0]);                          // m_mag
        m[3] = sqrtf(m[3]);                          // m_res
        float g[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) g[i] = robust_unit(m[i] + 0.0f, lohi[2 * i], lohi[2 * i + 1]);
        const float acc = fuse_score(p, g[0], g[1], g[2], g[3]);
        const size_t o = (size_t)b * Nv + tid;
        score[o] = acc;
        scores[tid] = acc != acc ? 0u : float_key(acc);          // NaN ranks lowest
        if (normed)
#pragma unroll
            for (int i = 0; i < 4; ++i) normed[i * ((size_t)B * Nv) + o] = g[i];
    }
    if (K < 0) return;
    const int k = K < Nv ? K : Nv;
    int32_t *out = keep_idx + (size_t)b * k;
    if (k == Nv && tid < Nv) out[tid] = tid;
    __syncthreads();
    if (k == 0 || k == Nv) return;
    if (wave == 0) {
        uint32_t key[WAVE_KEYS];
        wave_keys(Nv, key, [&](int i) { return scores[i]; });
        const uint32_t thr = wave_select(key, Nv, Nv - k, counters[0]);
        if (tid == 0) threshold = thr;
    }
    __syncthreads();
    // a wave's tokens above and at the threshold, behind those of the waves before it
    const uint32_t mine = scores[at], thr = threshold;
    const bool above = tid < Nv && mine > thr, ties = tid < Nv && mine == thr;
    const unsigned long long gt = __ballot(above), eq = __ballot(ties);
    if ((tid & 63) == 0) counts[wave] = __popcll(gt) << 16 | __popcll(eq);
    __syncthreads();
    const int n = (tid & 63) < SCORE_WAVES ? counts[tid & 63] : 0, upto = wave_incl_scan(n);
    const int before = __builtin_amdgcn_readlane(upto - n, wave), need = k - (__builtin_amdgcn_readlane(upto, 63) >> 16);
    const int g = count_before(gt, before >> 16), e = count_before(eq, before & 0xFFFF);
    if (above || (ties && e < need)) out[g + min(e, need)] = tid;          // (ties: lowest indices first)
}

// One wave per sequence of up to SCORE_THREADS tokens
__global__ __launch_bounds__(64) void small_topk_kernel(const float *__restrict__ score, int Nv, int K, int32_t *__restrict__ keep_idx)
{
    __shared__ __align__(16) int counters[256];
    const int b = blockIdx.x;
    int32_t *out = keep_idx + (size_t)b * K;
    if (K >= Nv) {          // host passes K <= Nv; K == Nv keeps every token
        for (int i = threadIdx.x; i < Nv; i += 64) out[i] = i;
        return;
    }
    uint32_t key[WAVE_KEYS];
    wave_keys(Nv, key, [&](int i) { return __float_as_uint(score[(size_t)b * Nv + i]); });
    for_keys(Nv, [&](int r) {
        const float f = __uint_as_float(key[r]);
        key[r] = f != f ? 0u : float_key(f);         // NaN ranks lowest
    });
    wave_topk(key, Nv, K, out, counters);
}

template <int PER>
__global__ __launch_bounds__(SCORE_THREADS) void topk_kernel(const float *__restrict__ score, int Nv, int K,
                                                             int32_t *__restrict__ keep_idx)
{
    __shared__ __align__(16) int hist[3 * 256];
    __shared__ uint32_t range[SELECT_RANGE];
    __shared__ int counts[2 * PER * SCORE_WAVES];
    const int b = blockIdx.x;
    int32_t *out = keep_idx + (size_t)b * K;
    if (K >= Nv) {          // host passes K <= Nv; K == Nv keeps every token
        for (int i = threadIdx.x; i < Nv; i += SCORE_THREADS) out[i] = i;
        return;
    }
    uint32_t key[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const float f = score[(size_t)b * Nv + min((int)threadIdx.x + SCORE_THREADS * r, Nv - 1)];
        key[r] = f != f ? 0u : float_key(f);          // NaN ranks lowest
    }
    topk_phase<PER>(key, Nv, K, out, hist, range, counts);
}

// Launches the score (+ top-k) kernel with the LDS its Nv needs: up to 153 KB at 8192 tokens, which
// is above the default limit of a launch and has to be granted once per device.
int launch_score_topk(const MetricSrc &src, long stride_sq, int B, int Nv, const quota_score_params &p,
                      float *score, float *normed, int K, int32_t *keep_idx, hipStream_t st, PrefetchList *weights = nullptr,
                      const quota_cue_masses *masses = nullptr, const quota_rows_beside *beside = nullptr)
{
    const auto share = weights ? weights->take(B, 7.0f, 4.0f) : PrefetchList::Share{};
    if (Nv <= SCORE_THREADS) {
        share.run([&](auto pre) {
            auto launch = [&](auto rows, int more) {
                const dim3 grid(B + more + share.wgs), block(SCORE_THREADS);
                auto with = [&](auto means) {
                    small_score_topk_kernel<<<grid, block, 0, st>>>(src.sumsq, src.ressq, src.cm_inter, src.cm_intra, B, Nv, K, (int)stride_sq, score, keep_idx,
                                                                    normed, p, means, pre, rows);
                };
                if (masses) with(*masses);
                else with(MeansThere{});
            };
            if (!beside) launch(NoRows{}, 0);
            else if (beside->d <= 4096) launch(RowsBeside<2>{*beside}, RowsBeside<2>{*beside}.wgs());
            else launch(RowsBeside<4>{*beside}, RowsBeside<4>{*beside}.wgs());
        });
        QUOTA_RETURN_IF_LAUNCH_FAILED();
        return QUOTA_OK;
    }
    const int cap = (Nv + 63) & ~63;
    const size_t lds = ((size_t)4 * cap + SELECT_HIST + SELECT_RANGE + 8) * sizeof(uint32_t);
    if (Nv > 2 * SCORE_THREADS) {          // the widest instantiations: up to 153 KB, above a launch's default 64 KB
        static bool granted[64];
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return QUOTA_ERR_HIP;
        if (!granted[dev]) {
            const size_t most = ((size_t)4 * MAXV + SELECT_HIST + SELECT_RANGE + 8) * sizeof(uint32_t);
            for (const void *k : {(const void *)score_topk_kernel<3, Prefetch>, (const void *)score_topk_kernel<3, NoPrefetch>,
                                  (const void *)score_topk_kernel<MAXV / SCORE_THREADS, Prefetch>,
                                  (const void *)score_topk_kernel<MAXV / SCORE_THREADS, NoPrefetch>})
                if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most) != hipSuccess)
                    return QUOTA_ERR_HIP;
            granted[dev] = true;
        }
    }
    share.run([&](auto pre) {
        using P = decltype(pre);
        auto kernel = Nv <= 3 * SCORE_THREADS ? score_topk_kernel<3, P> : score_topk_kernel<MAXV / SCORE_THREADS, P>;
        kernel<<<dim3(B + share.wgs), dim3(SCORE_THREADS), lds, st>>>(src, stride_sq, B, Nv, p, score, normed, K, keep_idx, cap, pre);
    });
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

int check_score_args(const float *sumsq, const float *ressq, const float *cm_inter,
                     const float *cm_intra, int B, int Nv, const quota_score_params *p, float *score)
{
    if (!sumsq || !ressq || !cm_inter || !cm_intra || !p || !score) return QUOTA_ERR_NULL;
    if (B <= 0 || Nv < 0 || p->pct_lo < 0 || p->pct_hi > 100 || p->pct_lo > p->pct_hi)
        return QUOTA_ERR_INVALID_ARG;
    if (Nv > MAXV) return QUOTA_ERR_SHAPE;
    return QUOTA_OK;
}

}  // namespace

int quota_internal_score(const float *sumsq, const float *ressq, long stride_sq,
                         const float *cm_inter, const float *cm_intra, int B, int Nv,
                         const quota_score_params *p, float *score, float *normed, hipStream_t st)
{
    int rc = check_score_args(sumsq, ressq, cm_inter, cm_intra, B, Nv, p, score);
    if (rc != QUOTA_OK) return rc;
    if (Nv == 0) return QUOTA_OK;
    ProfScope prof(QUOTA_K_SCORE_TOKENS, 0, 20.0 * B * Nv, st);
    MetricSrc src{sumsq, ressq, cm_inter, cm_intra, 0, 0};
    return launch_score_topk(src, stride_sq, B, Nv, *p, score, normed, -1, nullptr, st);
}

// Whether the kernel above makes the cues' head means itself: one CU then reads all masses of a sequence, at some 15 KB a us, where their
// own launch takes 2.4 us (8 heads) to 4.7.  Up to 80 KB it is ahead, one layer of a replayed stack, us less: 512 channels, 8 heads,
// 64 tokens 0.7, 256 0.8, 576 0.2; 7B shape, 32 heads, 101 tokens 3.2, 160 2.9, 256 1.7, 300 0.0, 320 -0.7, 576 -5.6; 13B shape, 40 heads, 250 tokens 1.3.
bool quota_score_takes_means(int Nv, int H) { return Nv <= SCORE_THREADS && (long)Nv * H <= 10240; }

// Rows to quantize beside it, four to a workgroup: up to 1024, one workgroup of 1024 threads a CU, are done before the tokens are scored.  A layer that so picks
// its rows against one that gathers them, replayed, us less (1024 rows in, kept share of the image 0.04 / 0.1 / 0.3 / 0.45): 4096 columns -0.1 / 0.5 / 1.5 / 2.8, 5120
// at 0.05 and 0.4 1.6 and 4.3, 8192 at 0.04 and 0.4 0.3 and 1.4, 512 1.7 and 2.1, 1024 1.5 and 2.9, 2048 1.1 and 2.4; 640 rows at 0.02 4096 columns 3.9, at 0.05 5120 2.7,
// 8192 3.3; 165 rows 2.8; 2 x 512 rows at 0.05 and 0.4 0.9 and 2.9, 8 x 128 at 0.2 -0.2.
bool quota_score_quantizes_beside(int Nv, int M, int d) { return Nv > 0 && Nv <= SCORE_THREADS && M > 0 && M <= 1024 && d % 128 == 0 && d <= 8192; }

// score + top-k in one launch (the layer's path)
int quota_internal_score_topk(const float *sumsq, const float *ressq, long stride_sq,
                              const float *cm_inter, const float *cm_intra, int B, int Nv,
                              const quota_score_params *p, float *score, int K, int32_t *keep_idx,
                              hipStream_t st, PrefetchList *weights, const quota_cue_masses *masses, const quota_rows_beside *beside)
{
    if (!sumsq || !ressq || !p || !score || !keep_idx || !cm_inter || !cm_intra) return QUOTA_ERR_NULL;
    if (B <= 0 || Nv < 0 || K < 0 || p->pct_lo < 0 || p->pct_hi > 100 || p->pct_lo > p->pct_hi)
        return QUOTA_ERR_INVALID_ARG;
    if (Nv > MAXV) return QUOTA_ERR_SHAPE;
    if (Nv == 0) return QUOTA_OK;
    if (masses && !quota_score_takes_means(Nv, masses->H)) return QUOTA_ERR_SHAPE;
    if (beside && !quota_score_quantizes_beside(Nv, beside->M, beside->d)) return QUOTA_ERR_SHAPE;
    ProfScope prof(QUOTA_K_SCORE_TOKENS, 0,
                   20.0 * B * Nv + 4.0 * B * (K < Nv ? K : Nv) + (beside ? 2.5 * beside->M * beside->d + 4.0 * beside->M : 0.0), st);
    MetricSrc src{sumsq, ressq, cm_inter, cm_intra, 0, 0};
    return launch_score_topk(src, stride_sq, B, Nv, *p, score, nullptr, K, keep_idx, st, weights, masses, beside);
}

extern "C" void quota_score_params_default(quota_score_params *p)
{
    if (!p) return;
    p->w_m = 0.25f; p->w_c = 0.45f; p->w_s = 0.10f; p->w_r = 0.20f;
    p->pct_lo = 10; p->pct_hi = 90;
}

extern "C" int quota_score_tokens(const float *sumsq, const float *ressq, const float *cm_inter,
                                  const float *cm_intra, int B, int Nv,
                                  const quota_score_params *p, float *score, float *normed_opt,
                                  void *stream)
{
    return quota_internal_score(sumsq, ressq, Nv, cm_inter, cm_intra, B, Nv, p, score, normed_opt,
                                (hipStream_t)stream);
}

extern "C" int quota_topk_prune(const float *score, int B, int Nv, int K, int32_t *keep_idx,
                                void *stream)
{
    if (!score || !keep_idx) return QUOTA_ERR_NULL;
    if (B <= 0 || Nv < 0 || K < 0) return QUOTA_ERR_INVALID_ARG;
    if (Nv > MAXV) return QUOTA_ERR_SHAPE;
    int k = K < Nv ? K : Nv;
    if (k == 0) return QUOTA_OK;
    ProfScope prof(QUOTA_K_TOPK_PRUNE, 0, 4.0 * B * Nv + 4.0 * B * k, (hipStream_t)stream);
    if (Nv <= SCORE_THREADS) small_topk_kernel<<<dim3(B), dim3(64), 0, (hipStream_t)stream>>>(score, Nv, k, keep_idx);
    else topk_kernel<MAXV / SCORE_THREADS><<<dim3(B), dim3(SCORE_THREADS), 0, (hipStream_t)stream>>>(score, Nv, k, keep_idx);
    QUOTA_RETURN_IF_LAUNCH_FAILED();
    return QUOTA_OK;
}

extern "C" int quota_score_tokens_from_hidden(const void *v_f16, int B, int Nv, int d, int ldv,
                                              long stride_b, const float *cm_inter,
                                              const float *cm_intra, const quota_score_params *p,
                                              float *score, float *normed_opt, void *ws,
                                              void *stream)
{
    if (!ws) return QUOTA_ERR_NULL;
    if (B <= 0 || Nv < 0) return QUOTA_ERR_INVALID_ARG;
    float *sumsq = (float *)ws, *ressq = sumsq + (size_t)B * Nv;
    int rc = quota_internal_vector_metrics(v_f16, B, Nv, d, ldv, stride_b, sumsq, ressq,
                                           (hipStream_t)stream);
    if (rc != QUOTA_OK) return rc;
    return quota_internal_score(sumsq, ressq, Nv, cm_inter, cm_intra, B, Nv, p, score, normed_opt,
                                (hipStream_t)stream);
}

extern "C" const char *quota_strerror(int code)
{
    switch (code) {
    case QUOTA_OK: return "ok";
    case QUOTA_ERR_NULL: return "a required pointer is null";
    case QUOTA_ERR_INVALID_ARG: return "invalid argument";
    case QUOTA_ERR_SHAPE: return "shape not supported by the kernels";
    case QUOTA_ERR_CAPACITY: return "KV cache or workspace capacity exceeded";
    case QUOTA_ERR_HIP: return "HIP runtime reported a launch error";
    default: return "unknown error code";
    }
}

extern "C" int quota_version(void) { return 100; }
