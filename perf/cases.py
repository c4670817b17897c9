"""The work a user of this package has it do, as cases that can be timed and compared.

A case is a plain dict; ``prepare`` builds what a program holds before the call (weights, caches,
descriptors, inputs -- all seeded, drawn on the device), ``run`` makes one pass through the public
classes of ``paper_2604_17320_amd.model``, ``work`` says what one pass cannot do without.

Kinds
  prefill      a pruned W4A4 prefill through 1..32 layers (PrefillStack.run), called eagerly or replayed
               from a HIP graph the program captured once
  decode       one decode step through 1..32 layers over their pruned 4-bit caches (PrefillStack.decode),
               eagerly or as the captured step of a decode loop
  sensitivity  Eq. 1's profile of one block on calibration samples (profile_sensitivity): the low-bit and the
               full-precision block on the same input
  pack         one projection on its way into the library: fp32 weights -> int4 codes and scales -> GEMM
               layout (PackedLinear.from_fp32)
"""
import torch

from paper_2604_17320_amd import binding as qb
from paper_2604_17320_amd import workloads as wl
from paper_2604_17320_amd.model import (FullPrecisionLayer, KVCache4, PackedLinear, PrefillLayer, PrefillStack,
                                        profile_sensitivity)

# language-model shapes of the workload configurations and of the grouped-query tests
MODELS = {
    "small": dict(d=512, H=8, Hkv=8, F=1376),
    "7b": dict(d=4096, H=32, Hkv=32, F=11008),
    "13b": dict(d=5120, H=40, Hkv=40, F=13824),
    "gqa": dict(d=3584, H=28, Hkv=4, F=18944),
}
NO_PRUNING = -1.0          # keep: a stack of layers outside the candidate set (qb.KEEP_ALL)


def _prefill(name, model, layers, B, before, Nv, after, keep, keep_last, graph):
    """keep: share of the Nv visual tokens left by the first pruning layer, falling linearly to keep_last at
    the last layer (stacks deeper than two layers keep everything in the first two)."""
    return dict(name=name, kind="prefill", model=model, layers=layers, B=B, before=before, Nv=Nv, after=after,
                keep=keep, keep_last=keep_last, graph=graph)


def _decode(name, model, layers, B, rows, rows_last, graph):
    """rows: cached tokens of the first layer, falling linearly to rows_last at the last one."""
    return dict(name=name, kind="decode", model=model, layers=layers, B=B, rows=rows, rows_last=rows_last,
                graph=graph)


def listed():
    return [
        # the smallest layer of the configurations: eleven dependent launches of a few microseconds each
        _prefill("prefill_small_layer", "small", 1, 1, 0, 64, 16, 0.3, 0.3, False),
        # the first pruning layer of a 7B prompt with one image: 640 tokens come in, 30 % of the image stays
        _prefill("prefill_7b_layer", "7b", 1, 1, 0, 576, 64, 0.3, 0.3, False),
        # a layer late in the same stack, where pruning has left an odd handful of tokens
        _prefill("prefill_7b_late_layer", "7b", 1, 1, 0, 101, 64, 0.95, 0.95, False),
        # the whole 7B stack on one image prompt, captured once and replayed: the headline workload
        _prefill("prefill_7b_stack", "7b", 32, 1, 0, 576, 64, 61 / 150, 0.1, True),
        # batched serving: 16 prompts through the first pruning layer
        _prefill("prefill_7b_batch16", "7b", 1, 16, 0, 576, 128, 61 / 150, 61 / 150, False),
        # high-resolution images on the 13B shape, four prompts of 2944 tokens
        _prefill("prefill_13b_hires", "13b", 1, 4, 0, 2880, 64, 0.266, 0.266, False),
        # grouped-query layer outside the candidate set, text before and after a ragged image
        _prefill("prefill_gqa_keep_all", "gqa", 1, 1, 14, 1023, 64, NO_PRUNING, NO_PRUNING, False),
        # one user's chat after a pruned prompt: one token through 32 layers, called layer by layer
        _decode("decode_7b_single", "7b", 32, 1, 640, 122, False),
        # the batched-serving decode loop: 16 sequences, the captured step replayed
        _decode("decode_7b_batch16", "7b", 32, 16, 704, 186, True),
        # a long conversation on the grouped-query shape: few K/V heads, thousands of cached tokens
        _decode("decode_gqa_long", "gqa", 1, 3, 4003, 4003, False),
        # offline allocation: one block profiled on two calibration samples
        dict(name="sensitivity_7b", kind="sensitivity", model="7b", B=2, N=640),
        # loading a checkpoint: the gate/up projection of the 7B shape
        dict(name="pack_7b_gate_up", kind="pack", N=22016, K=4096),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _drawn(rng):
    kind = rng.choice(["prefill"] * 5 + ["stack"] + ["decode"] * 4 + ["sensitivity", "pack"])
    model = rng.choice(["small", "7b", "7b", "13b", "gqa"])
    if kind in ("prefill", "stack"):
        layers = 1 if kind == "prefill" else _log(rng, 2, 32)
        keep = NO_PRUNING if rng.random() < 0.2 else rng.uniform(0.1, 0.9)
        last = keep if layers == 1 or keep < 0 else rng.uniform(0.05, keep)
        c = _prefill("", model, layers, _log(rng, 1, 16), rng.choice([0, 0, _log(rng, 1, 40)]), _log(rng, 32, 2880),
                     _log(rng, 8, 160), keep, last, layers > 1)
    elif kind == "decode":
        # whole stacks decode over pruned prompts; the long conversations come layer by layer
        layers = rng.choice([1, _log(rng, 2, 32)])
        rows = _log(rng, 16, 8000 if layers == 1 else 1000)
        c = _decode("", model, layers, _log(rng, 1, 32), rows, max(8, int(rows * rng.uniform(0.1, 1.0))),
                    rng.random() < 0.5)
    elif kind == "sensitivity":
        c = dict(kind=kind, model=model, B=_log(rng, 1, 8), N=_log(rng, 64, 1024))
    else:
        m = MODELS[model]
        N, K = rng.choice([(m["d"] + 2 * m["Hkv"] * (m["d"] // m["H"]), m["d"]), (m["d"], m["d"]),
                           (2 * m["F"], m["d"]), (m["d"], m["F"])])
        c = dict(kind=kind, N=N, K=K)
    c.pop("name", None)
    return c


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / 1e15


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _drawn(rng)
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------------------------- sizes

def _dims(model):
    m = MODELS[model]
    return m["d"], m["H"], m["Hkv"], m["d"] // m["H"], m["F"]


def _budgets(case):
    """Visual tokens each layer keeps (K_l)."""
    L, Nv = case["layers"], case["Nv"]
    if case["keep"] < 0:
        return [qb.KEEP_ALL] * L
    full = 2 if L > 2 else 0
    n = L - full
    ks = [Nv] * full
    for i in range(n):
        r = case["keep"] + (case["keep_last"] - case["keep"]) * (i / (n - 1) if n > 1 else 0.0)
        ks.append(max(1, -int(-(r * Nv) // 1)))
    return ks


def _cached_rows(case):
    L, a, b = case["layers"], case["rows"], case["rows_last"]
    return [int(round(a + (b - a) * (i / (L - 1) if L > 1 else 0.0))) for i in range(L)]


def _weight_bytes(model):
    d, H, Hkv, dh, F = _dims(model)
    n = (d + 2 * Hkv * dh) * d + d * d + 3 * d * F
    return n * (0.5 + 2 / 128), n


def work(case):
    if case["kind"] == "pack":
        n = case["N"] * case["K"]
        return {"bytes": 4.0 * n + n * (0.5 + 2 / 128), "flops": 2.0 * n}
    d, H, Hkv, dh, F = _dims(case["model"])
    dkv, B = Hkv * dh, case["B"]
    wbytes, wn = _weight_bytes(case["model"])
    qkv_n, rest_n = (d + 2 * dkv) * d, d * d + 3 * d * F
    row = dkv + dkv / 16                                   # K and V codes and scales of one cached token
    if case["kind"] == "prefill":
        N, Nv, by, fl = case["before"] + case["Nv"] + case["after"], case["Nv"], 0.0, 0.0
        by += B * N * (2 * d + 4)                          # the prompt's hidden state and positions
        for K in _budgets(case):
            k = Nv if K < 0 else min(K, Nv)
            n = N - Nv + k
            fl += 2.0 * B * N * qkv_n + 2.0 * B * n * rest_n + 4.0 * B * d * N * (N + 1) / 2
            if K >= 0:                                     # the visual keys' share of the attention matrix
                fl += 2.0 * B * d * (Nv * (N - case["before"]) - Nv * (Nv - 1) / 2)
            by += wbytes + B * n * row
            N, Nv = n, k
        return {"bytes": by + B * N * (2 * d + 4), "flops": fl}
    if case["kind"] == "decode":
        rows = _cached_rows(case)
        return {"bytes": len(rows) * wbytes + B * (sum(rows) + 2 * len(rows)) * row + 4.0 * B * d,
                "flops": 2.0 * B * len(rows) * wn + 4.0 * B * d * (sum(rows) + len(rows))}
    M = B * case["N"]
    attn = 4.0 * B * d * case["N"] * (case["N"] + 1) / 2
    return {"bytes": wbytes + 2.0 * wn + 2.0 * M * d + 16 * B, "flops": 2 * (2.0 * M * wn + attn)}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] == "sensitivity":
        return {"rel": 1e-3}               # norms of fp16 tensors: the roundings of single elements average out
    # fp16 tensors behind int4 quantizers: a last-place difference moves single values by a quantization step
    return {"rel": 1e-2, "differ": 1e-3}


# ------------------------------------------------------------------------------------ inputs

def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1009 + stream) % (2 ** 62))
    return g


def _matrices(model, seed, stream):
    """The four fp32 N(0, 0.02) projections of one layer, one after another."""
    d, H, Hkv, dh, F = _dims(model)
    g = _generator(seed, stream)
    for n, k in ((d + 2 * Hkv * dh, d), (d, d), (2 * F, d), (d, F)):
        yield torch.randn((n, k), generator=g, device="cuda") * 0.02


def _gains(model, seed, stream):
    g = _generator(seed, stream)
    return [torch.rand(_dims(model)[0], generator=g, device="cuda") + 0.5 for _ in range(2)]


def _hidden(model, rows, seed, stream):
    """fp16 N(0,1) with one channel in a hundred twenty times as large."""
    d = _dims(model)[0]
    g = _generator(seed, stream)
    x = torch.randn((rows, d), generator=g, device="cuda")
    x[:, torch.randperm(d, generator=g, device="cuda")[: max(1, d // 100)]] *= 20.0
    return x.to(torch.float16)


def _tables(model, n_pos):
    return [torch.from_numpy(t).cuda() for t in wl.rope_tables(_dims(model)[3], n_pos)]


def _layers(case, seed, n, n_pos):
    d, H, Hkv, dh, F = _dims(case["model"])
    cos, sin = _tables(case["model"], n_pos)
    out = []
    for i in range(n):
        w = [PackedLinear.from_fp32(m) for m in _matrices(case["model"], seed, 10 + 2 * i)]
        g1, g2 = _gains(case["model"], seed, 11 + 2 * i)
        out.append(PrefillLayer(H, dh, F, *w, g1, g2, 1e-5, cos, sin, Hkv))
    return out


def _one_arena(caches):
    """Puts the caches of a stack behind one another in four buffers, as a server keeps them."""
    arenas = []
    for kind in ("k_codes", "v_codes", "k_scales", "v_scales"):
        old = [getattr(c, kind) for c in caches]
        sizes = [-(-t.numel() // 128) * 128 for t in old]
        arena = torch.zeros(sum(sizes), dtype=old[0].dtype, device="cuda")
        at = 0
        for c, t, n in zip(caches, old, sizes):
            view = arena[at: at + t.numel()].view(t.shape)
            setattr(c, kind, view)
            setattr(c.desc, kind, view.data_ptr())
            at += n
        arenas.append(arena)
    return arenas


def _capture(call):
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    return graph, out


def _prepare_prefill(case, seed):
    N = case["before"] + case["Nv"] + case["after"]
    layers = _layers(case, seed, case["layers"], N)
    stack = PrefillStack(layers, case["B"], N, case["before"], case["Nv"], _budgets(case))
    s = dict(stack=stack, caches=_one_arena(stack.caches), x=_hidden(case["model"], case["B"] * N, seed, 1),
             pos=torch.arange(N, dtype=torch.int32, device="cuda").repeat(case["B"]))
    s["call"] = lambda: stack.run(s["x"], s["pos"])
    return s


def _prepare_decode(case, seed):
    d, H, Hkv, dh, F = _dims(case["model"])
    B, rows = case["B"], _cached_rows(case)
    layers = _layers(case, seed, case["layers"], max(rows) + 1)
    # a stack whose layers hold as many tokens as pruning left them
    stack = PrefillStack(layers, B, rows[0], 0, rows[0], [qb.KEEP_ALL] * len(rows), decode_capacity=16)
    stack.caches = [KVCache4(B, n + 16, Hkv, dh) for n in rows]
    arenas = _one_arena(stack.caches)
    for i, (c, n) in enumerate(zip(stack.caches, rows)):
        g = _generator(seed, 5000 + i)
        k, v = (torch.randn((B * n, Hkv * dh), generator=g, device="cuda").to(torch.float16) for _ in range(2))
        qb.quota_kv_quant_append(k, v, B, n, Hkv, dh, None, n, c.desc)
    s = dict(stack=stack, caches=arenas, x=_hidden(case["model"], B, seed, 1), rows=rows,
             pos=torch.full((B,), max(rows), dtype=torch.int32, device="cuda"))

    def step():
        if not case["graph"]:
            for c, n in zip(stack.caches, rows):       # every pass decodes the same token of the sequence
                c.desc.len = n
        return stack.decode(s["x"], s["pos"])
    if case["graph"]:
        stack.begin_stepped_decode(16)                 # the step count on the device, as a captured loop has it
    s["call"] = step
    return s


def prepare(case, seed):
    if case["kind"] == "pack":
        g = _generator(seed, 10)
        return dict(kind="pack", w=torch.randn((case["N"], case["K"]), generator=g, device="cuda") * 0.02)
    if case["kind"] == "sensitivity":
        d, H, Hkv, dh, F = _dims(case["model"])
        B, N = case["B"], case["N"]
        layer = _layers(case, seed, 1, N)[0]
        full = FullPrecisionLayer(H, dh, F, *_matrices(case["model"], seed, 10), layer.gamma1, layer.gamma2, 1e-5,
                                  layer.cosT, layer.sinT, Hkv)
        return dict(kind="sensitivity", layer=layer, full=full, B=B, N=N, x=_hidden(case["model"], B * N, seed, 1),
                    pos=torch.arange(N, dtype=torch.int32, device="cuda").repeat(B))
    s = (_prepare_prefill if case["kind"] == "prefill" else _prepare_decode)(case, seed)
    s["kind"] = case["kind"]
    if case["graph"]:
        s["replay"], s["out"] = _capture(s["call"])
    return s


def run(state):
    if state["kind"] == "pack":
        lin = PackedLinear.from_fp32(state["w"])
        return lin.packed, lin.scales
    if state["kind"] == "sensitivity":
        return profile_sensitivity(state["layer"], state["full"], state["x"], state["pos"], state["B"], state["N"])
    if "replay" in state:
        state["replay"].replay()
        out = state["out"]
    else:
        out = state["call"]()
    return out, state["caches"]
