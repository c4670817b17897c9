#!/usr/bin/env python3
"""Load-rate probe for gfx950: what a 16-byte load of all lanes (1 KB) costs a CU by the order of its addresses, from
global memory and from LDS.

Global: the addresses that the W4A4 GEMMs ask for, from 16 KB that a CU's own cache holds (what is left is the address unit)
and from 512 KB that every XCD's L2 holds.  `weights`: lane l takes piece
l / 16 of the 64 bytes of column l % 16, one contiguous KB in the order the products want; `rows`: 64 bytes of each of 16
rows that lie 33 lines apart, as activations do.  LDS: rows of 128 bytes whose 16-byte piece p sits at p ^ (r % 8),
read by 16 rows (W4A4 GEMM) or 32 (fp16 GEMM), beside the same unpermuted and consecutive addresses.

    python -m paper_2604_17320_amd.ubench.load_rate        # needs hipcc and a GPU
"""
import os
import subprocess
import sys
import tempfile

BUFFER = 1 << 20                       # bytes, a power of two
# byte of lane l (c = l % 16, q = l / 16); a load starts at a multiple of 1 KB in the window
GLOBAL = [("contiguous", "16 * l"), ("weights: 64 c + 16 q", "64 * c + 16 * q"), ("rows: 4224 c + 16 q", "4224 * c + 16 * q")]
# 16-byte piece of lane l (r = l % 32, h = l / 32); eight loads walk over 8 KB
LDS = [("consecutive", "l"), ("16 rows, permuted", "8 * c + ((2 * q) ^ (c & 7))"), ("32 rows, permuted", "8 * r + (h ^ (r & 7))"),
       ("32 rows, as they are", "8 * r + h")]

SOURCE = r'''
#include <hip/hip_runtime.h>
#include <cstdio>
template <int MODE>
__global__ __launch_bounds__(512) void global_loads(const char *buf, unsigned window, unsigned *out, int iters)
{
    const unsigned l = threadIdx.x & 63, c = l & 15, q = l >> 4;
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned at = 0, acc = 0;
    (void)c; (void)q;
@@GLOBAL@@
    for (int it = 0; it < iters; ++it) {
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            unsigned first = ((unsigned)(it * 8 + u) * 8 + wave) * 1024 & (window - 1);
            asm volatile("" : "+s"(first));
            v[u] = *reinterpret_cast<const uint4 *>(buf + first + at);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    out[blockIdx.x * blockDim.x + threadIdx.x] = acc;
}
template <int MODE>
__global__ __launch_bounds__(512) void lds_loads(unsigned *out, int iters)
{
    __shared__ uint4 lds[1024];
    for (int i = threadIdx.x; i < 1024; i += blockDim.x) lds[i] = make_uint4(i, i, i, i);
    __syncthreads();
    const unsigned l = threadIdx.x & 63, c = l & 15, q = l >> 4, r = l & 31, h = l >> 5;
    unsigned at = 0, acc = 0;
    (void)c; (void)q; (void)r; (void)h;
@@LDS@@
    for (int it = 0; it < iters; ++it) {
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            unsigned a = at;
            asm volatile("" : "+v"(a));
            v[u] = lds[(a ^ 2 * (u & 3)) + 256 * (u >> 2)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    out[blockIdx.x * blockDim.x + threadIdx.x] = acc;
}
template <typename F>
void time_it(const char *what, int waves, F launch)
{
    const int iters = 2000;
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0); (void)hipEventCreate(&e1);
    launch(100);
    (void)hipEventRecord(e0);
    launch(iters);
    (void)hipEventRecord(e1);
    (void)hipEventSynchronize(e1);
    float ms = 0.0f; (void)hipEventElapsedTime(&ms, e0, e1);
    printf("    %-24s %2d waves  %6.2f ns\n", what, waves, ms * 1e6f / (iters * 8.0f * waves));
}
int main()
{
    char *buf; unsigned *out;
    if (hipMalloc(&buf, @@BUFFER@@) != hipSuccess || hipMalloc(&out, 256 * 512 * 4) != hipSuccess) return 2;
    if (hipMemset(buf, 1, @@BUFFER@@) != hipSuccess) return 2;
    for (unsigned window : {16384u, @@BUFFER@@u / 2}) {
        printf("global, ns per KB of a CU (256 workgroups, one per CU), %u KB\n", window >> 10);
@@RUN_GLOBAL@@
    }
    printf("LDS, ns per KB of a CU\n");
@@RUN_LDS@@
    return hipDeviceSynchronize() == hipSuccess ? 0 : 3;
}
'''


def source():
    for _, at in GLOBAL:               # every address inside the buffer, every piece inside the 16 KB of LDS
        assert max(eval(at, dict(l=l, c=l % 16, q=l // 16)) for l in range(64)) + 16 + BUFFER // 2 - 1024 <= BUFFER
    for _, at in LDS:
        assert max(eval(at, dict(l=l, c=l % 16, q=l // 16, r=l % 32, h=l // 32)) | 7 for l in range(64)) + 256 < 1024
    pick = lambda cases: "\n".join(f"    if (MODE == {i}) at = {at};" for i, (_, at) in enumerate(cases))
    run = lambda cases, call: "\n".join(
        f'    for (int waves : {{4, 8}}) time_it("{what}", waves, [&](int n) {{ {call.format(i)}; }});' for i, (what, _) in enumerate(cases))
    s = SOURCE.replace("@@GLOBAL@@", pick(GLOBAL)).replace("@@LDS@@", pick(LDS)).replace("@@BUFFER@@", str(BUFFER))
    s = s.replace("@@RUN_GLOBAL@@", run(GLOBAL, "global_loads<{}><<<256, 64 * waves>>>(buf, window, out, n)"))
    return s.replace("@@RUN_LDS@@", run(LDS, "lds_loads<{}><<<256, 64 * waves>>>(out, n)"))


def main():
    with tempfile.TemporaryDirectory() as tmp:
        path, exe = os.path.join(tmp, "load_rate.hip"), os.path.join(tmp, "load_rate")
        with open(path, "w") as f:
            f.write(source())
        cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-Xclang", "-target-feature",
               "-Xclang", "-packed-fp32-ops", path, "-o", exe]
        done = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
        if done.returncode != 0:
            sys.exit(done.stderr)
        if "--build-only" in sys.argv:
            return 0
        return subprocess.run([exe]).returncode


if __name__ == "__main__":
    sys.exit(main())
