#!/usr/bin/env python3
"""Issue-rate probe for gfx950: what the matrix instruction of the W4A4 GEMM (v_mfma_f32_16x16x128_f8f6f4) and the
vector instructions that it needs beside it cost a SIMD, alone and interleaved, at one and two waves per SIMD.

A 128-channel group of a wave's RT x CT blocks of 16 x 16 outputs takes RT CT products of e2m3 numbers, 4 RT CT fp32
multiply-adds for the group's scale, 14 CT integer instructions that unpack its weights and, without start values, RT
products against the constant that removes the codes' offset.  This probe places exactly those mixes by hand (one asm block, fixed registers,
register-to-register only, no memory access in the timed loop, results meaningless) so that the compiler's scheduling is out
of the picture, and prints ns per group and the share of the matrix rate that the products alone reach.

    python -m paper_2604_17320_amd.ubench.issue_rate        # needs hipcc and a GPU
"""
import os
import subprocess
import sys
import tempfile

SHAPES = [("128 x 256 tile, wave 8 x 4 blocks", 8, 4), ("128 x 128, wave 8 x 2", 8, 2), ("64 x 128, wave 4 x 2", 4, 2),
          ("32 x 128, wave 2 x 2", 2, 2), ("32 x 64, wave 2 x 1", 2, 1)]

TEMPLATE = r'''
#include <hip/hip_runtime.h>
#include <cstdio>
template <int MODE>
__global__ __launch_bounds__(256) void k(float *out, int iters)
{
    float s = threadIdx.x;
#pragma unroll 1
    for (int it = 0; it < iters; ++it) {
@@CASES@@
    }
    out[blockIdx.x * 256 + threadIdx.x] = s;
}
template <int MODE>
float run(float *d, int wgs)
{
    const int iters = 4000;
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0); (void)hipEventCreate(&e1);
    k<MODE><<<wgs, 256>>>(d, 10);
    (void)hipDeviceSynchronize();
    (void)hipEventRecord(e0);
    k<MODE><<<wgs, 256>>>(d, iters);
    (void)hipEventRecord(e1);
    (void)hipEventSynchronize(e1);
    float ms = 0.0f; (void)hipEventElapsedTime(&ms, e0, e1);
    return ms * 1e6f / iters;
}
int main()
{
    float *d;
    if (hipMalloc(&d, 4096 * 256 * 4) != hipSuccess) return 2;
    for (int wgs : {256, 512}) {
        printf("%d wave(s) per SIMD: ns per group (of each wave), and the products alone against it\n", wgs / 256);
@@RUNS@@
    }
    return 0;
}
'''

MFMA, FMA, UNPACK = "mfma", "fma", "unpack"


def mix(rt, ct, offset, scale, unpack):
    """The instructions of a group, vector work spread evenly behind the matrix instructions."""
    mats = rt * ct + (rt if offset else 0)
    vec = [FMA] * (4 * rt * ct if scale else 0) + [UNPACK] * (14 * ct if unpack else 0)
    order, done = [], 0
    for m in range(mats):
        order.append(MFMA)
        upto = len(vec) * (m + 1) // mats
        order += vec[done:upto]
        done = upto
    return order


def block(order):
    lines, m, f, u = [], 0, 0, 0
    for what in order:
        if what == MFMA:                                   # eight results take turns; the chain reads one four places back
            a = 64 + 4 * (m % 8)
            lines.append(f"v_mfma_f32_16x16x128_f8f6f4 v[{a}:{a + 3}], v[160:165], v[168:173], v[96:99] cbsz:2 blgp:2")
            m += 1
        elif what == FMA:
            lines.append(f"v_fmac_f32_e32 v{100 + f % 48}, v{64 + (4 * (m + 3) + f) % 32}, v148")
            f += 1
        else:
            reg, other = 150 + u % 8, 150 + (u + 3) % 8
            lines.append(f"v_alignbit_b32 v{reg}, v{reg}, v{other}, 30" if u % 7 == 0 else
                         f"v_bitop3_b32 v{reg}, v{reg}, v{other}, v148 bitop3:{'0x6a' if u % 2 else '0x78'}")
            u += 1
    return "\\n\\t".join(lines)


def main():
    cases, runs, mode = [], [], 0
    clobber = ",".join(f'"v{i}"' for i in range(64, 176))
    for name, rt, ct in SHAPES:
        steps = [("products", (False, False, False)), ("+ scale chain", (False, True, False)),
                 ("+ unpack: with start values", (False, True, True)), ("+ offset products: without", (True, True, True))]
        runs.append(f'        {{ float t, t0 = 0; (void)t0; printf("  {name}\\n");')
        for i, (what, flags) in enumerate(steps):
            cases.append(f'        {"else " if mode else ""}if (MODE == {mode}) asm volatile("{block(mix(rt, ct, *flags))}" ::: {clobber});')
            keep = " t0 = t;" if i == 0 else ""
            runs.append(f'        t = run<{mode}>(d, wgs);{keep} printf("    %-28s %8.1f ns   %5.1f %%\\n", "{what}", t, 100 * t0 / t);')
            mode += 1
        runs.append("        }")
    src = TEMPLATE.replace("@@CASES@@", "\n".join(cases)).replace("@@RUNS@@", "\n".join(runs))
    with tempfile.TemporaryDirectory() as tmp:
        path, exe = os.path.join(tmp, "issue_rate.hip"), os.path.join(tmp, "issue_rate")
        with open(path, "w") as f:
            f.write(src)
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
