// A layer's weights on their way from HBM into the last-level cache (256 MB, behind the L2s) while its short kernels leave
// CUs and memory idle.  Attention, cues and top-k of a short prompt run on a few workgroups for 7 to 18 us each; workgroups
// beyond theirs read the scales and weights of the O, gate/up and down projections, in the order of their use, and drop them.  The
// projections then wait for that cache instead of HBM, stage after stage: 32 layers of 7B, 640 to 122 tokens, each layer's weights used
// once, 4709 -> 4430 us (gate/up 30.3 -> 28.0, O and down together 35.0 -> 31.6, attention and cues 1 us longer each);
// one layer over changing weights, 640 tokens 166 -> 158, 165 tokens 127 -> 124.  Scales first: without them every stage
// waits for HBM as before (4590).
#pragma once
#include "common.h"

struct Prefetch {                       // up to six ranges of 16-byte pieces
    static constexpr int RANGES = 6;
    const uint4 *at[RANGES];
    unsigned n[RANGES];
};

// What a launch without a share takes in its place: the kernel is then another, without these workgroups' code and 72 bytes of
// arguments, which cost the host 3 us a launch when its caches are cold (first pass of a layer of 512 channels 125 -> 116 us, 115 before
// there was anything to fetch).
struct NoPrefetch {};
template <int NT>
__device__ __forceinline__ void prefetch(const NoPrefetch &, int, int) {}

// Workgroup `wg` of `wgs` reads its share, 8 pieces a thread in flight.
template <int NT>
__device__ __forceinline__ void prefetch(const Prefetch &p, int wg, int wgs)
{
    for (int r = 0; r < Prefetch::RANGES; ++r) {
        const unsigned n = p.n[r];
        for (unsigned first = (unsigned)wg * (8 * NT); first < n; first += (unsigned)wgs * (8 * NT)) {
            uint4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p.at[r][min(first + NT * u + threadIdx.x, n - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
        }
    }
}

// What is still to be fetched; a launch takes what fits beside it.
class PrefetchList {
    Prefetch left = {};
    int ranges = 0;
    size_t total = 0;                                  // pieces

public:
    void add(const void *p, size_t bytes)              // (whole 16-byte pieces, at their multiples)
    {
        const uintptr_t a = ((uintptr_t)p + 15) & ~(uintptr_t)15, e = (uintptr_t)p + bytes;
        left.at[ranges] = (const uint4 *)a;
        left.n[ranges] = e > a ? (unsigned)((e - a) / 16) : 0;
        total += left.n[ranges++];
    }
    // For a launch of `wgs` workgroups that lasts for about `us`: what `rate` MB a microsecond bring in that time, and the
    // workgroups to bring it, 128 KB each at least.  Only where a quarter of the CUs is idle: beside 252 workgroups a GQA layer of 1101
    // tokens over changing weights takes 314 us instead of 299, beside 3072 the longer ones gain nothing (4 x 2944 tokens
    // 1966 -> 1981).  Less than 4 MB in all (a layer of 512 channels) are not worth the workgroups: 51.9 us without, 52.7 with.
    struct Share {
        Prefetch what;
        unsigned wgs;
        template <typename LAUNCH> void run(LAUNCH launch) const
        {
            if (wgs) launch(what);
            else launch(NoPrefetch{});
        }
    };
    Share take(unsigned wgs, float us, float rate)
    {
        Share s = {};
        if (wgs > 192 || total < (4u << 16)) return s;
        unsigned room = (unsigned)(us * rate * 65536.0f), all = 0;
        for (int r = 0; r < ranges; ++r) {
            const unsigned n = left.n[r] < room ? left.n[r] : room;
            s.what.at[r] = left.at[r];
            s.what.n[r] = n;
            left.at[r] += n;
            left.n[r] -= n;
            room -= n;
            all += n;
        }
        const unsigned most = (all + 8191) / 8192;
        s.wgs = most < 256 - wgs ? most : 256 - wgs;
        return s;
    }
};
