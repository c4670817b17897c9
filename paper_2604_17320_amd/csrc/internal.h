// Host-side launchers shared between translation units of libquota (not part
// of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include "../../include/quota.h"
#include "prefetch.h"
#include "headmeans.h"

// The rows that a layer keeps, [B][n_keep] of [B][N]: text before the visual tokens, the kept ones of those, text behind.
struct quota_kept_rows {
    const int32_t *keep_idx;
    int N, vis_begin, Nv, k_keep, n_keep;
    // The index that row j of sequence b needs (k_keep > 0, keep_idx given; row j of the text reads one that it does not need), and with it the row of the
    // sequence: never one outside it
    __device__ __forceinline__ int index(int b, int j) const { return keep_idx[(size_t)b * k_keep + min(max(j - vis_begin, 0), k_keep - 1)]; }
    __device__ __forceinline__ int row(int j, int idx) const
    {
        const int src = j < vis_begin ? j : j < vis_begin + k_keep ? vis_begin + idx : j - k_keep + Nv;
        return min(max(src, 0), N - 1);
    }
};
// Rows to quantize beside a launch that leaves CUs idle: fp16 [M][d] into the A6 format without start values.
struct quota_rows_beside {
    const f16 *x;
    uint32_t *q;
    float *scale;
    int M, d;
};
// What is left of the compaction where nobody gathers rows: the kept rows' 4-bit K/V into the cache, their positions and numbers.
struct quota_kept_copies {
    quota_kept_rows kept;
    int rows, dkv, capacity, len;                // rows: of all sequences
    const uint32_t *skc, *svc;
    const f16 *sks, *svs;
    const int32_t *pos;
    uint32_t *ckc, *cvc;
    f16 *cks, *cvs;
    int32_t *pos_out, *rows_out;
};

// score kernel with a separate sequence stride for the sumsq/ressq arrays, so
// the layer can pass the per-row side outputs of the quantizer directly
int quota_internal_score(const float *sumsq, const float *ressq, long stride_sq,
                         const float *cm_inter, const float *cm_intra, int B, int Nv,
                         const quota_score_params *p, float *score, float *normed, hipStream_t st);

// score + top-k of the min(K, Nv) best tokens in one launch.  masses: the cues' head means are made there too, in the place
// of cm_inter and cm_intra, and left where it says; only where quota_score_takes_means allows it.
int quota_internal_score_topk(const float *sumsq, const float *ressq, long stride_sq,
                              const float *cm_inter, const float *cm_intra, int B, int Nv,
                              const quota_score_params *p, float *score, int K, int32_t *keep_idx,
                              hipStream_t st, PrefetchList *weights, const quota_cue_masses *masses, const quota_rows_beside *beside = nullptr);
bool quota_score_takes_means(int Nv, int H);
// Whether it takes rows to quantize beside it
bool quota_score_quantizes_beside(int Nv, int M, int d);

// attention and, if cm_inter or cm_intra is given, the cue pass with its head means [B][Nv]; masses: without the means, for whom they are
// left then
int quota_internal_attention(const void *q_f16, const void *khat_f16, const void *vhat_f16, int B,
                             int N, int H, int Hkv, int dh, int vis_begin, int Nv, void *o_f16,
                             float *cm_inter, float *cm_intra, void *ws, hipStream_t st, PrefetchList *weights,
                             quota_cue_masses *masses);

struct quota_compact_args {
    int B, N, vis_begin, Nv, k_keep, n_keep, d, dkv;      // dkv: width of a K or V row (Hkv * dh)
    const int32_t *keep_idx;              // null: the first k_keep visual tokens (k_keep = Nv: all of them)
    const void *x, *o;
    const int32_t *pos;
    const void *skc, *sks, *svc, *svs;     // staged 4-bit K/V of all N rows
    void *x_out, *o_out;                   // o_out optional (fp16 copy of the kept attention rows)
    uint8_t *oq_out;                       // optional: int4 codes of the kept attention rows (A6 format) ...
    float *os_out;                         // ... and their per-token scales (the quantizer Q)
    int32_t *pos_out, *rows_out;
    quota_kv_cache *cache;
};
// Appends at row cache->len but does not advance it.
int quota_internal_compact(const quota_compact_args *a, hipStream_t st);

int quota_internal_vector_metrics(const void *v_f16, int B, int Nv, int d, int ldv, long stride_b,
                                  float *sumsq, float *ressq, hipStream_t st);

// Decode attention of one new token per sequence straight from its QKV projection [B][d + 2 dkv]: RoPE, 4-bit K/V
// of the new row (appended at row cache->len, + *step_dev; len does not move), attention over the grown cache.
// part: quota_internal_decode_part_bytes bytes.
size_t quota_internal_decode_part_bytes(int B, int H, int Hkv, int dh);
int quota_internal_attention_decode_new(const void *qkv_f16, const int32_t *pos, const float *cosT, const float *sinT,
                                        int n_pos, int Hq, const quota_kv_cache *cache, void *q_rot_opt, void *o_f16,
                                        void *part, hipStream_t st);

// Arguments of the fused QKV epilogue: what quota_rope_kv_quant takes, minus the qkv input.
struct quota_qkv_epilogue {
    const int32_t *pos;
    const float *cosT, *sinT;
    int n_pos, d, dkv, dh;                  // q width H*dh, K/V width Hkv*dh
    f16 *q_rot, *khat, *vhat;
    uint32_t *k_codes, *v_codes;
    f16 *k_scales, *v_scales;
};
int quota_internal_w4a4_gemm_qkv(const uint8_t *qa6, const float *sa, int M, const quota_weights *W,
                                 void *y_opt, const quota_qkv_epilogue *qe, hipStream_t st);

// The layer's row quantizers and GEMM on activations in the A6 format (gemm.hip): four rows at a time, quota_a6_row_bytes(K)
// bytes for each (padded to whole fours), then, if quota_a6_starts(M), [groups][M] floats.
// (groups of a row in memory: stages of up to 8 groups may read past the last)
__host__ __device__ inline int quota_a6_groups(int G) { return ((G + 7) & ~7) | 1; }
inline size_t quota_a6_row_bytes(int K) { return (size_t)quota_a6_groups((K + 127) / 128) * 96; }
// The sums cost the quantizers more than the GEMMs gain where those wait for memory anyway.  Pairs of whole layers by a line at 256, 512, 1024
// and 2048 rows, us: 512 channels 78 to 198 at 270 to 2900 rows, within 1 % of each other; 7B shape 270 rows 259, 256, 256, 257, 640 rows 353, 351,
// 356, 357, 1800 rows 835, 835, 834, 822, but 800 rows 463, 465, 430, 433; 13B shape 530 rows 522, 527, 492, 488, 800 rows 624, 621, 631, 633, 1800
// rows 1153, 1156, 1152, 1182: not one line for all.
inline bool quota_a6_starts(size_t M) { return M >= 512; }
// Bytes of M rows in it, or as the few-row GEMM's fragments (up to 32 rows, 1 KB a group and 16 rows).
inline size_t quota_a6_bytes(size_t M, int K)
{
    const size_t G = ((size_t)K + 127) / 128, rows = (M + 3) / 4 * 4 * quota_a6_row_bytes(K);
    const size_t frag = M <= 32 ? (M + 15) / 16 * G * 1024 : 0;
    return (rows > frag ? rows : frag) + (quota_a6_starts(M) ? M * G * sizeof(float) : 0);
}
int quota_internal_rmsnorm_quantize_a6(const void *x_f16, int M, int d, const float *gamma, float eps, uint8_t *qa6,
                                       float *scale, float *sumsq_opt, float *ressq_opt, hipStream_t st, const quota_kept_copies *copies = nullptr);
int quota_internal_silu_mul_quantize_a6(const void *gu_f16, int M, int F, uint8_t *qa6, float *scale, void *z_opt,
                                        const void *z_inject_opt, hipStream_t st);
int quota_internal_quantize_a6(const void *x_f16, int M, int d, uint8_t *qa6, float *scale, hipStream_t st);
int quota_internal_w4a4_gemm_a6(const uint8_t *qa6, const float *sa, int M, const quota_weights *W, void *y_f16, int ldy,
                                const void *residual_opt, int ldr, hipStream_t st);
// The same on the kept rows of activations and residual, M of B * N: M > 16, below quota_a6_starts, scales on dwords (quota_gemm_gathers)
bool quota_gemm_gathers(int M, const quota_weights *W);
int quota_internal_w4a4_gemm_a6_kept(const uint8_t *qa6, const float *sa, int M, const quota_kept_rows *kept, const quota_weights *W, void *y_f16, int ldy,
                                     const void *residual, int ldr, hipStream_t st);
int quota_internal_w4a4_gemm_silu(const uint8_t *qa6, const float *sa, int M, const quota_weights *W, void *z_f16, hipStream_t st);

// GEMM of at most 16 rows, or as fragments 32 (rows16.hip).  The quantizing forms take fp16 rows, for the M and K that
// quota_internal_rows16_quantizes accepts: as they are, or through RMSNorm.  frag_silu and glu: the gate/up projection,
// z [M][N / 2] = SiLU(gate) * up.
enum quota_rows16_format { QUOTA_ROWS16_A6, QUOTA_ROWS16_PACKED, QUOTA_ROWS16_FRAG };
int quota_internal_rows16(const uint8_t *qa, quota_rows16_format format, const float *sa, int M, const quota_weights *W, void *y, int ldy,
                          const void *res, int ldr, hipStream_t st);
int quota_internal_rows16_frag_silu(const uint8_t *qf, const float *sa, int M, const quota_weights *W, void *z, hipStream_t st);
int quota_internal_rmsnorm_quantize_frag(const void *x_f16, int M, int d, const float *gamma, float eps, uint8_t *qf,
                                         float *scale, hipStream_t st);
int quota_internal_quantize_frag(const void *x_f16, int M, int d, uint8_t *qf, float *scale, hipStream_t st);
bool quota_internal_rows16_quantizes(int M, int K);
int quota_internal_rows16_quantize(const void *x, int M, const quota_weights *W, void *y, int ldy, const void *res,
                                   int ldr, hipStream_t st);
int quota_internal_rows16_rmsnorm(const void *x, const float *gamma, float eps, int M, const quota_weights *W, void *y,
                                  int ldy, bool glu, hipStream_t st);

// quota_rope_kv_quant with Hkv K/V heads: qkv rows are q (H*dh) | k (Hkv*dh) | v (Hkv*dh).
int quota_internal_rope_kv_quant(const void *qkv_f16, int M, int H, int Hkv, int dh, const int32_t *pos,
                                 const float *cosT, const float *sinT, int n_pos, void *q_rot_f16,
                                 void *khat_f16, void *vhat_f16, uint8_t *k_codes, void *k_scales,
                                 uint8_t *v_codes, void *v_scales, hipStream_t st);

// A workspace may start anywhere: its parts lie behind the first multiple of 16 (asynchronous copies read them), so that
// it holds QUOTA_WS_SLACK bytes more than they take.
#define QUOTA_WS_SLACK 16
inline char *quota_ws_start(void *ws) { return (char *)(((uintptr_t)ws + 15) & ~(uintptr_t)15); }

// *step_dev += 1 (one thread; capturable)
int quota_internal_advance_step(int32_t *step_dev, hipStream_t st);


// Limits that the kernels behind the layer calls enforce, for the up-front checks of the layer
// calls (a call that returns an error must not have enqueued anything).
#define QUOTA_MAX_SCORED_TOKENS 8192      // visual tokens per sequence the score / top-k kernel holds in LDS
#define QUOTA_MAX_DECODE_ROWS 8192        // cached rows per sequence the decode attention softmaxes over
#define QUOTA_MAX_MODEL_WIDTH 16384       // d: the compaction gather keeps a row in registers
#define QUOTA_MAX_ROW_COLS 32768          // widest row of the row quantizers (the FFN width F)
