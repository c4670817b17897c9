// A layer's weights on their way from HBM into the last-level cache (256 MB, behind the L2s) while its short kernels leave
// CUs and memory idle.  Attention, cues and top-k of a short prompt run on a few workgroups for 7 to 18 us each; workgroups
// beyond theirs read the scales and weights of the O, gate/up and down projections, in the order of their use, and drop them.  The
// projections then wait for that cache instead of HBM, stage after stage: 32 layers of 7B, 640 to 122 tokens, each layer's weights used
// once, 4710 -> 4505 us (gate/up 30.3 -> 28.0, O and down together 35.0 -> 31.6, attention and cues 1 us longer each);
// one layer over changing weights, 640 tokens 164.7 -> 159.6, 165 tokens 125.7 -> 122.5.  Scales first: without them every stage
// waits for HBM as before (4590, and 4430 with them, on the same card).
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
    // Whether a layer of so many rows gains by it.  The launches of 128 rows or less are over before the bytes are there, and those of
    // less than 512 before less than 8 MB repay the workgroups (without -> with: stacks of 7B layers, 42 rows 693 -> 719 us, 80 rows within 1 %, 165
    // rows 1004 -> 986; 20 layers of 2048 channels, 19 MB each, 42 rows 1214 -> 1275, 165 rows 1582 -> 1525; 64 layers of 1024 channels, 5 MB,
    // 42 rows 3135 -> 3391, 300 rows 1 % more, 640 rows 4570 -> 4531).  Less than 4 MB never do (a layer of 512 channels 51.9 -> 52.7).
    bool worth(size_t rows) const { return rows > 128 && total >= (size_t)(rows < 512 ? 8 : 4) << 16; }
    // For a launch of `wgs` workgroups that lasts for about `us`: what `rate` MB a microsecond bring in that time, and the
    // workgroups to bring it, 128 KB each at most while CUs are left.  Only where a quarter of them is idle: beside 252 workgroups a GQA layer of 1101
    // tokens over changing weights takes 314 us instead of 299, beside 3072 the longer ones gain nothing (4 x 2944 tokens
    // 1966 -> 1981).
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
        if (wgs > 192) return s;
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
