// Head means of the attention cues, by whoever takes them: a launch of its own (attn.hip) or the workgroup that
// scores the sequence (select.hip).
#pragma once
#include "common.h"

// Per-head masses of the cue pass, [B][H][Nv] pairs (from text queries, from visual ones), and where their means [B][Nv] belong.
struct quota_cue_masses {
    const float2 *partial;
    int H;
    float *cm_inter, *cm_intra;
};

// The sums of both masses of key i of a sequence, by a quad of lanes (hq: which of it): lane hq sums heads [hq H/4 .. ) in head order, the
// four sums are combined as (s0 + s1) + (s2 + s3).  All lanes of the quad get them.
__device__ __forceinline__ float2 head_sums(const float2 *__restrict__ partial, int H, int Nv, int i, int hq)
{
    const int hper = (H + 3) / 4, h_lo = hq * hper, h_hi = min(h_lo + hper, H);
    const float2 *pp = partial + min(i, Nv - 1);
    float st = 0.0f, sv = 0.0f;
    for (int k0 = 0; k0 < hper; k0 += 8) {           // (uniform: lanes of a quad differ in their first head only)
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u < hper) v[u] = pp[(size_t)min(h_lo + k0 + u, H - 1) * Nv];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u < h_hi - h_lo) {
                st += v[u].x;
                sv += v[u].y;
            }
    }
    st += __shfl_xor(st, 1, 64); sv += __shfl_xor(sv, 1, 64);
    st += __shfl_xor(st, 2, 64); sv += __shfl_xor(sv, 2, 64);
    return make_float2(st, sv);
}
