"""GPU parity of the decode layer's own paths against the oracle: the attention that appends the new row while it
walks a cache of several tiles (one head or two per workgroup, whole or split over workgroups, called with a host-side
length or with the step count on the device), and the few-row GEMMs at every row count where their path changes.

Teacher-forced as in test_gpu_decode: with the oracle's attention output and SwiGLU product injected every integer and
fp16 tensor must be bit-exact, and the library's own attention output, dumped by the same run, is within 1e-2.  What lies
behind the cached rows, and the workspace, hold NaN bit patterns: nothing there may reach a result."""
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2604_17320_amd import workloads as wl
from test_gpu_ops import _pack4, close_f16, dev, host, unpack4
from test_gpu_decode import eq16, random_cache
from test_gpu_gqa import build_gqa_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    assert torch.cuda.is_available()
    from paper_2604_17320_amd import binding
    binding.lib()
    return binding


@functools.lru_cache(maxsize=2)
def layer(H, Hkv, dh, F):
    return build_gqa_layer(H * dh, H, Hkv, dh, F, 40, 64)


def poisoned_cache(c, B, rows, capacity, Hkv, dh):
    """A cache with `rows` of the oracle's rows; every byte behind them 0xFF (codes -1, scales NaN)."""
    from paper_2604_17320_amd.model import KVCache4
    cache = KVCache4(B, capacity, Hkv, dh)
    for t in (cache.k_codes, cache.v_codes, cache.k_scales, cache.v_scales):
        t.view(torch.uint8).fill_(0xFF)
    cache.k_codes[:, :rows], cache.v_codes[:, :rows] = dev(_pack4(c["kc"])), dev(_pack4(c["vc"]))
    cache.k_scales[:, :rows], cache.v_scales[:, :rows] = dev(c["ks"]), dev(c["vs"])
    cache.desc.len = rows
    return cache


def step_and_check(H, Hkv, dh, F, B, rows, stepped=None):
    """One decode step over `rows` cached rows.  stepped: (steps already taken, most steps of the loop)."""
    from paper_2604_17320_amd.model import make_taps
    W, L, cos, sin = layer(H, Hkv, dh, F)
    d, dkv = H * dh, Hkv * dh
    c = random_cache(rows, B, rows, Hkv, dh)
    r = wl.rng(rows, "decode-paths", B)
    x, pos = r.standard_normal((B, d)).astype(np.float16), (7 + np.arange(B) % 50).astype(np.int32)
    ref = oracle.decode_layer(W, x, pos, c, cos, sin)
    room = rows + 3 if stepped is None else rows - stepped[0] + stepped[1] + 3
    cache = poisoned_cache(c, B, rows, room, Hkv, dh)
    if stepped is not None:
        step_dev = torch.full((1,), stepped[0], dtype=torch.int32, device="cuda")
        cache.desc.len, cache.desc.step_dev, cache.desc.max_steps = rows - stepped[0], step_dev.data_ptr(), stepped[1]
    t16 = lambda *s: torch.full(s, float("nan"), dtype=torch.float16, device="cuda")
    out = dict(qkv=t16(B, d + 2 * dkv), q_rot=t16(B, d), o=t16(B, d), x1=t16(B, d), gu=t16(B, 2 * F))
    inject = dict(inject_o=dev(ref["o"]), inject_z=dev(ref["z"]))
    y = t16(B, d)
    ws = torch.full((L.decode_workspace_bytes(B),), 0xFF, dtype=torch.uint8, device="cuda")
    xd, pd = dev(x), dev(pos)
    L.decode(xd, pd, cache, y, ws, make_taps(**out, **inject))
    assert cache.len == (rows + 1 if stepped is None else rows - stepped[0])
    assert eq16(host(out["qkv"]), ref["qkv"]) and eq16(host(out["q_rot"]), ref["q"])
    kc, vc, ks, vs = (host(t) for t in (cache.k_codes, cache.v_codes, cache.k_scales, cache.v_scales))
    assert np.array_equal(unpack4(kc[:, rows]), ref["kc"]) and np.array_equal(unpack4(vc[:, rows]), ref["vc"])
    assert eq16(ks[:, rows], ref["ks"]) and eq16(vs[:, rows], ref["vs"])
    assert np.array_equal(kc[:, :rows], _pack4(c["kc"])) and np.array_equal(vc[:, :rows], _pack4(c["vc"]))
    assert eq16(ks[:, :rows], c["ks"]) and eq16(vs[:, :rows], c["vs"])
    for t in (kc, vc, ks.view(np.uint8), vs.view(np.uint8)):
        assert np.all(t[:, rows + 1:] == 0xFF)                  # nothing written behind the new row
    assert close_f16(host(out["o"]), ref["o"])
    assert eq16(host(out["x1"]), ref["x1"]) and eq16(host(out["gu"]), ref["gu"]) and eq16(host(y), ref["x_next"])


HEADS = [(8, 8, 64), (4, 4, 128), (8, 2, 128), (6, 2, 64)]      # rep 1 and 4; an odd group of 3 query heads


@pytest.mark.parametrize("H,Hkv,dh", HEADS)
@pytest.mark.parametrize("rows", [511, 512, 700, 1023,          # one to two 512-row tiles: the new row last and first in a tile
                                  1024, 1535, 2049, 3000,       # split over workgroups, one tile each
                                  5200])                        # into more than eight parts
def test_decode_layer_walks_and_splits(qb, H, Hkv, dh, rows):
    print(f"decode layer, {H}/{Hkv} heads of {dh}, {rows} cached rows", flush=True)
    step_and_check(H, Hkv, dh, 160, 2, rows)


@pytest.mark.parametrize("H,Hkv,dh", HEADS)
@pytest.mark.parametrize("rows,step,most", [(700, 3, 60),       # length on the device, unsplit
                                            (1200, 0, 40), (1536, 17, 400),     # split, new row in the last part
                                            (603, 3, 2400)])    # split for the longest loop: most parts have no rows yet
def test_decode_layer_stepped(qb, H, Hkv, dh, rows, step, most):
    print(f"stepped decode layer, {H}/{Hkv} heads of {dh}, {rows} cached rows, step {step} of {most}", flush=True)
    step_and_check(H, Hkv, dh, 160, 2, rows, (step, most))


@pytest.mark.parametrize("stepped", [None, (2, 30)])
@pytest.mark.parametrize("H,Hkv,dh,B,rows", [
    (32, 32, 64, 16, 511), (32, 32, 64, 16, 1100),              # two heads per workgroup, one tile and three
    (16, 16, 128, 32, 512), (16, 16, 128, 32, 640),
    (8, 8, 64, 12, 2900),                                       # parts of three tiles: a split that walks
    (8, 4, 128, 20, 2100),
])
def test_decode_layer_many_heads(qb, H, Hkv, dh, B, rows, stepped):
    print(f"decode layer, {H}/{Hkv} heads of {dh}, {B} sequences of {rows} cached rows, stepped {stepped}", flush=True)
    step_and_check(H, Hkv, dh, 160, B, rows, stepped)


@pytest.mark.parametrize("H,Hkv,dh,B,rows,most", [
    (8, 8, 64, 2, 700, 1000), (4, 4, 128, 2, 1020, 600), (8, 2, 128, 2, 1023, 400),     # one part, in loops that end in parts
    (8, 8, 64, 12, 1300, 2000),                                 # too few tiles to split, in a loop that ends in parts of two
    (8, 8, 64, 12, 2900, 2100), (8, 4, 128, 20, 2100, 1500),    # parts that grow within the loop
])
def test_decode_layer_stepped_has_the_eager_bits(qb, H, Hkv, dh, B, rows, most):
    """How the cached rows are split over workgroups, hence the order of the sums, depends on the rows there are and not on
    the loop's length: a step whose count lies on the device leaves the bits of the call with a host-side length."""
    from paper_2604_17320_amd.model import make_taps
    print(f"decode layer, {H}/{Hkv} heads of {dh}, {B} sequences of {rows} cached rows, eager and fourth of {most}", flush=True)
    W, L, cos, sin = layer(H, Hkv, dh, 160)
    c = random_cache(rows, B, rows, Hkv, dh)
    r = wl.rng(rows, "decode-eager", B)
    x, pos = dev(r.standard_normal((B, H * dh)).astype(np.float16)), dev((7 + np.arange(B) % 50).astype(np.int32))
    got = []
    for stepped in (False, True):
        cache, n = poisoned_cache(c, B, rows, rows + most, Hkv, dh), torch.full((1,), 3, dtype=torch.int32, device="cuda")
        if stepped:
            cache.desc.len, cache.desc.step_dev, cache.desc.max_steps = rows - 3, n.data_ptr(), most
        o, y = (torch.full((B, H * dh), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
        ws = torch.full((L.decode_workspace_bytes(B),), 0xFF, dtype=torch.uint8, device="cuda")
        L.decode(x, pos, cache, y, ws, make_taps(o=o))
        got.append((host(o), host(y)))
    assert np.isfinite(got[0][0].astype(np.float32)).all()
    assert eq16(got[0][0], got[1][0]) and eq16(got[0][1], got[1][1])


@pytest.mark.parametrize("F", [1376, 2720, 8736])      # gate/up 2752, 5440, 17472 columns; ragged rows into down, one of them long
@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 7, 11, 15, 16, 17, 32, 33, 70])
def test_decode_layer_row_counts(qb, F, B):
    """Up to 4 rows the GEMM quantizes its input, up to 16 it reads fragments of which it owns B rows, up to 32 two blocks of
    them; beyond that the projections go through the tiles.  (Down, behind the taps, reads rows of bytes.)"""
    print(f"decode layer, {B} rows, F = {F}", flush=True)
    step_and_check(8, 2, 64, F, B, 20)


@pytest.mark.parametrize("H,Hkv", [(32, 32), (48, 12), (64, 1)])       # QKV of 12288 x 4096, 9216 x 6144, 8448 x 8192
@pytest.mark.parametrize("B", [1, 2, 3])
def test_decode_layer_one_share_of_the_projection_per_cu(qb, H, Hkv, B):
    """One or two rows of at most three chunks per thread: a workgroup takes 48 columns where those are at most 256 shares.
    Beyond them it takes 32."""
    print(f"decode layer, {B} rows, {H}/{Hkv} heads of 128", flush=True)
    step_and_check(H, Hkv, 128, 160, B, 20)


@pytest.mark.parametrize("H,Hkv,dh,rows,most", [(8, 8, 64, 509, 8), (8, 2, 128, 1021, 1500)])
def test_decode_layer_captured_across_a_tile_boundary(qb, H, Hkv, dh, rows, most):
    """One captured step replayed while the cache grows past a 512-row tile (and, split, past a workgroup's share): every
    replay leaves the bits of the eager stepped call, and the caches end equal."""
    B, F, steps = 2, 160, 8
    _, L, _, _ = layer(H, Hkv, dh, F)
    c = random_cache(rows, B, rows, Hkv, dh)
    xs = dev(wl.rng(rows, "captured").standard_normal((steps, B, H * dh)).astype(np.float16))
    pos = torch.zeros(B, dtype=torch.int32, device="cuda")
    ws = torch.empty(L.decode_workspace_bytes(B), dtype=torch.uint8, device="cuda")
    eager, replayed = [], []
    caches, counters = [], []
    for _ in range(2):
        cache, n = poisoned_cache(c, B, rows, rows + most, Hkv, dh), torch.zeros(1, dtype=torch.int32, device="cuda")
        cache.desc.step_dev, cache.desc.max_steps = n.data_ptr(), most
        caches.append(cache)
        counters.append(n)
    y, x_in = torch.empty_like(xs[0]), torch.empty_like(xs[0])
    for i in range(steps):
        L.decode(xs[i], pos, caches[0], y, ws)
        qb.quota_advance_step(counters[0])
        eager.append(host(y).copy())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        L.decode(x_in, pos, caches[1], y, ws)
        qb.quota_advance_step(counters[1])
    for i in range(steps):
        x_in.copy_(xs[i])
        graph.replay()
        replayed.append(host(y).copy())
    assert int(counters[0]) == int(counters[1]) == steps
    assert all(eq16(a, b) for a, b in zip(eager, replayed))
    for name in ("k_codes", "v_codes", "k_scales", "v_scales"):
        a, b = (getattr(k, name)[:, : rows + steps].contiguous().view(torch.uint8) for k in caches)
        assert torch.equal(a, b), name


@pytest.mark.parametrize("F", [96, 1376, 2720, 4128, 8736])  # gate/up of 192 to 17472 columns: both widths of a workgroup's share
@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 7, 11, 15, 16, 17, 32, 33])
def test_decode_layer_silu_product_in_the_gate_up_projection(qb, F, B):
    """Without taps on gate | up or z the projection makes the product itself and down reads it as fragments or
    quantizes it: the bits of the step whose tap keeps the two kernels apart and whose down reads rows of bytes."""
    from paper_2604_17320_amd.model import make_taps
    H, Hkv, dh, rows = 8, 2, 64, 20
    W, L, cos, sin = layer(H, Hkv, dh, F)
    c = random_cache(rows, B, rows, Hkv, dh)
    r = wl.rng(F, "decode-silu", B)
    x, pos = dev(r.standard_normal((B, H * dh)).astype(np.float16)), dev((7 + np.arange(B) % 50).astype(np.int32))
    outs = []
    for taps in (dict(gu=torch.empty((B, 2 * F), dtype=torch.float16, device="cuda")), {}):
        cache = poisoned_cache(c, B, rows, rows + 1, Hkv, dh)
        y = torch.full((B, H * dh), float("nan"), dtype=torch.float16, device="cuda")
        ws = torch.full((L.decode_workspace_bytes(B),), 0xFF, dtype=torch.uint8, device="cuda")
        L.decode(x, pos, cache, y, ws, make_taps(**taps))
        outs.append(host(y))
    assert np.isfinite(outs[0].astype(np.float32)).all() and eq16(outs[0], outs[1])


@pytest.mark.parametrize("H,Hkv,dh,B", [(8, 8, 128, 1), (4, 4, 64, 16),      # V's channels by four workgroups, one query head and pairs
                                        (8, 2, 128, 4), (7, 1, 64, 16), (6, 2, 128, 20), (28, 4, 64, 8)])   # and by two
@pytest.mark.parametrize("rows", [1, 4, 127, 128, 511, 512, 700, 1023])      # ends of passes and tiles
def test_decode_layer_shared_channels_of_v_have_the_same_bits(qb, H, Hkv, dh, B, rows):
    """How many workgroups share a head's V is no matter of its sums: the layer's attention leaves the bits of a call on the
    rotated queries and the appended cache, whose workgroups own a head each."""
    from paper_2604_17320_amd.model import make_taps
    print(f"decode layer, {H}/{Hkv} heads of {dh}, {B} sequences of {rows} cached rows", flush=True)
    W, L, cos, sin = layer(H, Hkv, dh, 160)
    c = random_cache(rows, B, rows, Hkv, dh)
    r = wl.rng(rows, "decode-shared", B)
    x, pos = dev(r.standard_normal((B, H * dh)).astype(np.float16)), dev((7 + np.arange(B) % 50).astype(np.int32))
    cache = poisoned_cache(c, B, rows, rows + 2, Hkv, dh)
    q, o, y, whole = (torch.full((B, H * dh), float("nan"), dtype=torch.float16, device="cuda") for _ in range(4))
    ws = torch.full((L.decode_workspace_bytes(B),), 0xFF, dtype=torch.uint8, device="cuda")
    L.decode(x, pos, cache, y, ws, make_taps(q_rot=q, o=o))
    assert cache.len == rows + 1
    qb.quota_attention_decode_gqa(q, H, cache.desc, whole)
    assert np.isfinite(host(o).astype(np.float32)).all() and eq16(host(o), host(whole))
