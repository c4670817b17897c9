"""CPU checks of the host-side helpers that hold no method arithmetic: the synthetic workload
definitions (shapes, the keep schedules the benchmark and the stack tests run) and the tool that
condenses profiler CSVs into the summaries under profiles/."""
import csv
import glob
import os
import re
import struct
import subprocess
import sys

import msgpack
import numpy as np

from paper_2604_17320_amd import profile_summary as ps, workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_config_shapes():
    c1, c2, c3 = wl.CONFIGS[0], wl.CONFIGS[1], wl.CONFIGS[2]
    assert (c1.d, c1.H, c1.dh, c1.F, c1.N) == (512, 8, 64, 1376, 80)
    for c in (c2, c3):
        assert (c.d, c.H, c.dh, c.F, c.Nv, c.Nt) == (4096, 32, 128, 11008, 576, 64)
    assert c3.layers == 32 and c3.B == 1


def test_stack_schedule_is_the_stated_ramp():
    """Full budget on the first two layers, then the linear ramp that ends at 0.1 and averages 0.30
    over the 32 layers; ceil of exact rationals."""
    K = wl.schedule_for(wl.CONFIGS[2])
    assert K[:6] == [576, 576, 235, 229, 223, 216] and K[-4:] == [76, 70, 64, 58] and len(K) == 32
    assert all(a >= b for a, b in zip(K, K[1:]))
    assert abs(sum(K) / (32 * 576) - 0.3008) < 2e-4
    assert wl.schedule_for(wl.CONFIGS[1]) == [173]              # ceil(0.3 * 576), Table 4's operating point


def test_generators_are_seeded_and_shaped():
    s = wl.CONFIGS[0]
    x = wl.hidden_state(s, 3)
    assert x.dtype == np.float16 and x.shape == (s.B * s.N, s.d)
    assert np.array_equal(x, wl.hidden_state(s, 3)) and not np.array_equal(x, wl.hidden_state(s, 4))
    col_rms = np.sqrt((x.astype(np.float32) ** 2).mean(axis=0))
    assert (col_rms > 10).sum() == s.n_outlier                  # the outlier channels, and only they
    cos, sin = wl.rope_tables(64, 16)
    assert cos.shape == (16, 32) and np.allclose(cos ** 2 + sin ** 2, 1.0, atol=1e-6) and np.all(cos[0] == 1.0)


def test_profile_summary_classifies_library_kernels():
    f8 = "_ZN12_GLOBAL__N_114w4a4_f8_kernelILi%dELi%dELi%dELi%dELi%dELb%dELb%dELb%dELi2EEEvPKh"
    assert ps.classify(f8 % (4, 4, 2, 2, 6, 0, 0, 1)) == "w4a4_gemm_64x128"
    assert ps.classify(f8 % (4, 4, 2, 2, 6, 1, 1, 0)) == "w4a4_gemm_other"
    assert ps.classify(f8 % (2, 1, 4, 4, 0, 0, 0, 0)) == "w4a4_gemm_32x64"
    assert ps.classify("_ZN12_GLOBAL__N_118w4a4_rows16_kernelILi2ELi1ELi2ELi1EEEvNS_6RowsInE") == "w4a4_gemm_rows16"
    assert ps.classify("_Z27rmsnorm_quantize_act_kernelILb0ELi64ELi8EEv") == "rmsnorm_quantize_act"
    assert ps.classify("_Z19quantize_act_kernelILb1ELi64ELi8EEv") == "quantize_act"
    assert ps.bandwidth_case("_Z19quantize_act_kernelILb1ELi64ELi8EEv") == "quantize_act (+ m_mag, m_res)"
    assert ps.bandwidth_case("_Z27rmsnorm_quantize_act_kernelILb0ELi64ELi8EEv") == "rmsnorm_quantize_act"
    assert ps.classify("void at::native::elementwise_kernel<...>") is None


def test_profile_summary_knows_the_kernels_there_are():
    """Every kernel of the sources has a class, every class a kernel, and the classes that the library times
    carry the library's names."""
    names = set()
    for path in glob.glob(os.path.join(ROOT, "paper_2604_17320_amd", "csrc", "*.hip")):
        with open(path) as f:
            for head in re.findall(r"__global__(.*?)\{", f.read(), re.S):
                names.add(re.search(r"\b(\w+_kernel)\s*\(", head).group(1))
    mangled = {n: ps.classify(f"_ZN12_GLOBAL__N_1{len(n)}{n}EPKh") for n in names}
    unknown = {n for n, cls in mangled.items() if cls is None}
    assert unknown == {"empty_kernel", "w4a4_f8_kernel"}                       # (the latter: by its template arguments)
    assert {re.match(r"\w+?_kernel", key).group(0) for key, _ in ps.CLASSES} == names - {"empty_kernel"}
    gemm = set()
    with open(os.path.join(ROOT, "paper_2604_17320_amd", "csrc", "gemm.hip")) as f:
        for args in re.findall(r"#define F8_TILE_\d\(P, A, QK\)\s*w4a4_f8_kernel<([^>]*)>", f.read()):
            v = [a.strip() for a in args.split(",")]
            gemm.add(ps.classify("w4a4_f8_kernelI" + "".join(f"Li{a}E" if a.isdigit() else "Lb0E" for a in v)))
    assert len(gemm) == 5 and None not in gemm
    from paper_2604_17320_amd import binding
    timed = {binding.quota_kernel_name(i) for i in range(binding.KERNEL_COUNT)}
    assert gemm | {"w4a4_gemm_other", "w4a4_gemm_rows16", "attention_decode", "score_tokens", "pack_weights"} <= timed


def test_profile_summary_classes_of_the_built_gemm_tiles():
    """The class of every GEMM tile by the name that it has in the library: by rows and columns, and the one with the integer sums apart."""
    from paper_2604_17320_amd import binding
    with open(binding.LIB_PATH, "rb") as f:
        names = {m.decode() for m in re.findall(rb"_ZN12_GLOBAL__N_114w4a4_f8_kernel\w+", f.read())}
    seen = set()
    for name in names:
        rt, ct, nw, sums = map(int, re.search(r"ILi(\d+)ELi(\d+)ELi(\d+)E.*?ActFormatE\dELb(\d)E", name).groups())
        want = "w4a4_gemm_other" if sums else f"w4a4_gemm_{16 * rt}x{16 * ct * nw}"
        assert ps.classify(name) == want, name
        seen.add(want)
    assert seen == {"w4a4_gemm_other"} | {f"w4a4_gemm_{t}" for t in ("128x128", "64x128", "32x128", "32x64", "128x256", "64x256")}


def kernel_resources(path):
    """{kernel name: its metadata} of the gfx950 code objects inside a library built here."""
    with open(path, "rb") as f:
        data = f.read()
    kernels = {}
    for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", data):                       # (0x40: the AMD HSA ABI)
        elf = data[m.start():]
        at, size, n = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
        for i in range(n):
            kind, = struct.unpack_from("<I", elf, at + size * i + 4)
            first, length = struct.unpack_from("<QQ", elf, at + size * i + 24)
            while kind == 7 and length >= 12:                                       # notes
                name, desc, note = struct.unpack_from("<III", elf, first)
                body = first + 12 + (name + 3 & ~3)
                if note == 32:                                                      # AMDGPU metadata
                    for k in msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]:
                        kernels[k[".name"]] = k
                step = 12 + (name + 3 & ~3) + (desc + 3 & ~3)
                first, length = first + step, length - step
    return kernels


def workgroups_per_cu(k):
    """Resident workgroups of four waves, one per SIMD: 512 registers a lane of a SIMD in eights, 160 KB of LDS."""
    by_registers = min(8, 512 // (k[".vgpr_count"] + 7 & ~7))
    lds = k[".group_segment_fixed_size"]
    return min(by_registers, 160 * 1024 // lds)


def test_gemm_tiles_leave_room_for_the_workgroups_that_their_choice_counts_on():
    """The choice of a tile goes by times that were measured with so many of its workgroups on a CU: one fewer, for a few registers more, and
    launches of more workgroups take a fifth longer."""
    from paper_2604_17320_amd import binding
    room = {"8ELi2": 3, "4ELi2": 3, "2ELi2": 3, "2ELi1": 5, "8ELi4": 2, "6ELi2": 2}         # a layer's rows; row and column blocks of a wave
    packed = {"8ELi2": 2, "4ELi2": 3, "2ELi2": 3, "2ELi1": 4, "8ELi4": 2, "4ELi4": 2}
    seen = set()
    for name, k in kernel_resources(binding.LIB_PATH).items():
        m = re.search(r"w4a4_(?:f8|rows96)_kernelILi(\d+ELi\d+)ELi4ELi(\d+)E\w*?ActFormatE(\d)E", name)
        if not m:
            continue
        blocks, stage, acts = m.groups()
        want = packed[blocks] if acts == "2" else 3 if (blocks, stage) == ("2ELi1", "8") else room[blocks]
        assert workgroups_per_cu(k) >= want, (name, k[".vgpr_count"], k[".group_segment_fixed_size"])
        seen.add((blocks, acts == "2"))
    assert seen == {(b, False) for b in room} | {(b, True) for b in packed}


def test_gemm_keeps_a_table_of_rows_only_where_it_picks_them():
    """The tiles that pick rows have LDS for their rows' numbers, the others of a layer's rows none."""
    from paper_2604_17320_amd import binding
    lds = {}
    for name, k in kernel_resources(binding.LIB_PATH).items():
        m = re.search(r"w4a4_\w+_kernelI(Li(\d+)E(?:Li\d+E)*).*?ActFormatE0ELb0ELNS_8EpilogueE(\d)E", name)
        if m:
            lds.setdefault((m.group(1), 16 * int(m.group(2))), {})[int(m.group(3))] = k[".group_segment_fixed_size"]
    picked = {tile: by for tile, by in lds.items() if 3 in by}
    assert len(picked) == 7                                                    # every tile that a layer's rows can take
    for (tile, rows), by in picked.items():
        assert by[3] >= by[0] + 4 * rows, tile


def test_few_row_gemm_loads_residuals_only_where_they_are_added():
    """Whether there are residuals is an argument of the kernel's template: packed rows, A6 rows and fragments come both ways,
    rows quantized in the launch only with them, normalised ones and gate/up only without."""
    from paper_2604_17320_amd import binding
    by_mode = {}
    for name in kernel_resources(binding.LIB_PATH):
        m = re.search(r"w4a4_rows16_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)ELi(\d)ELb(\d)E", name)
        assert m or "w4a4_rows16" not in name, name
        if m:
            nb, u, mode, nc, glu, rb, res = map(int, m.groups())
            by_mode.setdefault((mode, glu, nb, u, nc, rb), set()).add(res)
    assert {k[:2] for k in by_mode} == {(0, 0), (1, 0), (2, 0), (2, 1), (3, 0), (4, 0), (4, 1)}       # A6, packed, fragments, quantizing, RMSNorm
    for (mode, glu, *_), res in by_mode.items():
        assert res == ({0} if glu or mode == 4 else {1} if mode == 3 else {0, 1}), (mode, glu, res)


def test_profile_summary_stats_table(tmp_path, capsys):
    rows = [dict(Name="_Z19quantize_act_kernelILb0ELi64ELi8EEv", Calls=4, TotalDurationNs=100000),
            dict(Name="_ZN12_GLOBAL__N_115attn_fwd_kernelILi128EEEv", Calls=2, TotalDurationNs=30000),
            dict(Name="some_other_kernel", Calls=9, TotalDurationNs=999)]
    p = tmp_path / "stats.csv"
    with open(p, "w", newline="") as f:
        w = csv.DictWriter(f, fieldnames=["Name", "Calls", "TotalDurationNs"])
        w.writeheader()
        w.writerows(rows)
    ps.stats(str(p))
    out = capsys.readouterr().out
    assert "quantize_act" in out and "25.00" in out and "attention_fwd" in out and "15.00" in out
    assert "some_other_kernel" not in out


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode == 2 and "ONE GPU" in r.stderr and r.stdout.strip() == ""
