"""GPU parity of quota_prefill_layer against the oracle's layer composite.

Two modes.  Teacher-forced: the oracle's attention output, column masses and
SwiGLU product are injected at the library's tap points, so every integer
output and every fp16 tensor downstream must then be BIT-EXACT.  Free-running:
the GPU consumes its own floats; fp16 tensors must be within 1e-2 relative,
scores within 1e-5 relative (after the column masses' own tolerance), and the
kept index set must equal the oracle's except where the oracle's score gap
across the cut is below that tolerance."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17320_amd import workloads as wl
from test_gpu_ops import close_f16, dev, host, unpack4

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    assert torch.cuda.is_available()
    from paper_2604_17320_amd import binding
    binding.lib()
    return binding


def build_layer(shape, seed, gamma_random=False):
    from paper_2604_17320_amd.model import PackedLinear, PrefillLayer
    fw = wl.fp_weights(shape, seed)
    q = {k: oracle.quantize_weights(v) for k, v in fw.items()}
    d = shape.d
    if gamma_random:
        g1 = wl.rng(seed, "g1").uniform(0.7, 1.3, d).astype(np.float32)
        g2 = wl.rng(seed, "g2").uniform(0.7, 1.3, d).astype(np.float32)
    else:
        g1 = np.ones(d, np.float32)
        g2 = np.ones(d, np.float32)
    W = oracle.LayerWeights(qkv=q["qkv"], o=q["o"], gu=q["gu"], down=q["down"], gamma1=g1, gamma2=g2,
                            eps=1e-5, H=shape.H, dh=shape.dh, F=shape.F)
    cos, sin = wl.rope_tables(shape.dh, shape.N + 8)
    lin = {k: PackedLinear.from_codes(dev(c), dev(s)) for k, (c, s) in q.items()}
    L = PrefillLayer(shape.H, shape.dh, shape.F, lin["qkv"], lin["o"], lin["gu"], lin["down"], dev(g1),
                     dev(g2), 1e-5, dev(cos), dev(sin))
    return W, L, cos, sin


def run_gpu(qb, L, shape, x, pos, K, inject=None):
    from paper_2604_17320_amd.model import KVCache4, make_taps
    B, N, Nv, vb, d, F = shape.B, shape.N, shape.Nv, shape.vis_begin, shape.d, shape.F
    k = min(K, Nv)
    n_keep = N - Nv + k
    t = lambda shp, dt: torch.zeros(shp, dtype=dt, device="cuda")
    out = dict(qkv=t((B * N, 3 * d), torch.float16), q_rot=t((B * N, d), torch.float16),
               o=t((B * N, d), torch.float16), sumsq=t((B, max(Nv, 1)), torch.float32),
               ressq=t((B, max(Nv, 1)), torch.float32), cm_inter=t((B, max(Nv, 1)), torch.float32),
               cm_intra=t((B, max(Nv, 1)), torch.float32), score=t((B, max(Nv, 1)), torch.float32),
               keep_idx=t((B, max(k, 1)), torch.int32), rows=t((B, max(n_keep, 1)), torch.int32),
               x1=t((max(B * n_keep, 1), d), torch.float16), gu=t((max(B * n_keep, 1), 2 * F), torch.float16),
               z=t((max(B * n_keep, 1), F), torch.float16))
    keep_alive = []
    taps = dict(out)
    if inject:
        for name, arr in inject.items():
            tens = dev(arr)
            keep_alive.append(tens)
            taps["inject_" + name] = tens
    cache = KVCache4(B, n_keep + 3, shape.H, shape.dh)
    x_out = t((max(B * n_keep, 1), d), torch.float16)
    pos_out = t((max(B * n_keep, 1),), torch.int32)
    ws = torch.empty(L.workspace_bytes(B, N), dtype=torch.uint8, device="cuda")
    xd, pd = dev(x), dev(pos)
    st = qb.State(B, N, vb, Nv, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, make_taps(**taps), ws)
    res = {k_: host(v) for k_, v in out.items()}
    res.update(x_next=host(x_out), pos_next=host(pos_out), N=st.N, Nv=st.Nv, cache_len=cache.len,
               cache_kc=unpack4(host(cache.k_codes)[:, :n_keep]).reshape(B * n_keep, d),
               cache_vc=unpack4(host(cache.v_codes)[:, :n_keep]).reshape(B * n_keep, d),
               cache_ks=host(cache.k_scales)[:, :n_keep].reshape(B * n_keep, -1),
               cache_vs=host(cache.v_scales)[:, :n_keep].reshape(B * n_keep, -1))
    return res


def assert_teacher_forced_exact(ref, got, shape, K):
    B, Nv = shape.B, shape.Nv
    k = min(K, Nv)
    n_keep = shape.N - Nv + k
    eq16 = lambda a, b: np.array_equal(np.ascontiguousarray(a).view(np.uint16), np.ascontiguousarray(b).view(np.uint16))
    assert eq16(got["qkv"], ref["qkv"]) and eq16(got["q_rot"], ref["q"])
    if Nv:
        assert np.array_equal(got["sumsq"], ref["sumsq"]) and np.array_equal(got["ressq"], ref["ressq"])
        assert np.array_equal(got["score"], ref["score"])
    assert got["N"] == n_keep and got["Nv"] == k and got["cache_len"] == n_keep
    if k:
        assert np.array_equal(got["keep_idx"][:, :k], ref["keep_idx"])
    if n_keep:
        assert np.array_equal(got["rows"], ref["rows"])
        assert np.array_equal(got["pos_next"][: B * n_keep], ref["pos_next"])
        assert np.array_equal(got["cache_kc"], ref["cache_kc"]) and np.array_equal(got["cache_vc"], ref["cache_vc"])
        assert eq16(got["cache_ks"], ref["cache_ks"]) and eq16(got["cache_vs"], ref["cache_vs"])
        assert eq16(got["x1"], ref["x1"]) and eq16(got["gu"], ref["gu"])
        assert eq16(got["x_next"][: B * n_keep], ref["x_next"])


CASES = [
    # name, shape overrides, K
    ("c1", dict(), 19),
    ("many_rows", dict(B=8, Nv=384, Nt=16), 100),      # 3200 rows: the tile choices of mid-sized launches
    ("c1_k20", dict(), 20),
    ("keep_all", dict(), 999),
    ("keep_none", dict(), 0),
    ("batch2_prefix", dict(B=2, vis_begin=3, Nt=9), 19),
    ("no_visual", dict(Nv=0, Nt=40), 5),
    ("one_row_left", dict(Nt=1), 0),                   # rows behind the compaction: the few-row GEMM quantizes its input,
    ("three_rows_left", dict(Nt=2), 1),
    ("nine_rows_left", dict(B=3, Nt=2), 1),            # reads fragments of 9 and 15 rows,
    ("fifteen_rows_left", dict(Nt=9), 6),
    ("seventeen_rows_left", dict(Nt=9), 8),            # and gives way to the tiles
    ("long_visual_prefix", dict(Nv=4100, Nt=28), 1000),   # more scored tokens than fit the default LDS limit of a launch
]


@pytest.mark.parametrize("name,over,K", CASES, ids=[c[0] for c in CASES])
def test_layer_small_teacher_forced(qb, name, over, K):
    base = wl.CONFIGS[0]
    kw = dict(name=name, d=base.d, H=base.H, F=base.F, layers=1, B=base.B, Nv=base.Nv, Nt=base.Nt,
              n_outlier=base.n_outlier, vis_begin=0)
    kw.update(over)
    shape = wl.Shape(**kw)
    W, L, cos, sin = build_layer(shape, 0, gamma_random=True)
    x, pos = wl.hidden_state(shape, 0), wl.positions(shape)
    ref = oracle.prefill_layer(W, x, pos, shape.B, shape.N, shape.vis_begin, shape.Nv, K, cos, sin,
                               prune_mid=True)
    inject = dict(o=ref["o"], z=ref["z"])
    if shape.Nv:
        inject.update(cm_inter=ref["cm_inter"], cm_intra=ref["cm_intra"])
    got = run_gpu(qb, L, shape, x, pos, K, inject)
    assert_teacher_forced_exact(ref, got, shape, K)
    # the GPU's own attention / cue / SwiGLU outputs, dumped by the same run, within tolerance
    assert close_f16(got["o"], ref["o"])
    if shape.Nv:
        assert np.allclose(got["cm_inter"], ref["cm_inter"], rtol=2e-5, atol=1e-7)
        assert np.allclose(got["cm_intra"], ref["cm_intra"], rtol=2e-5, atol=1e-7)


def close_f32(a, b, rtol=1e-5):
    """fp32 contract: |a - b| <= rtol * max(|b|, rms(b)), element by element."""
    a, b = a.astype(np.float64), b.astype(np.float64)
    rms = np.sqrt((b ** 2).mean()) if b.size else 0.0
    return bool(np.all(np.abs(a - b) <= rtol * np.maximum(np.abs(b), rms)))


# Share of int4 codes that may differ at a quantizer of a free-running chain.  A code flips when the
# two sides' inputs fall on different sides of a rounding boundary: inputs that differ by one fp16
# ulp (2^-11 relative) do so with probability ~ |x| / step * 2^-11 per element (a few 1e-3 at most);
# a row whose absmax element moved re-scales the whole row, which moves more codes of that row.
# Flips then feed the next quantizer through an exact GEMM and a row normalisation or a product.
FLIP_BOUND = dict(qa2=2e-3, qa3=2e-3, qa4=5e-3)      # measured: up to 3.3e-4, 1e-5, 8.5e-4


def free_running_report(ref, got, shape, K, W):
    """Where a free-running GPU chain and the oracle part ways, quantizer by quantizer: the int4
    codes each quantizer WOULD emit for the GPU's tensor (oracle quantizer applied to it -- the GPU
    quantizers equal it bit for bit on equal inputs) against the oracle's own codes.  Rows are the
    kept rows common to both sides."""
    B, N, Nv = shape.B, shape.N, shape.Nv
    k = min(K, Nv)
    n_keep = N - Nv + k
    g_rows, r_rows = got["rows"].reshape(B, n_keep), ref["rows"].reshape(B, n_keep)
    gi, ri = [], []                                    # positions (in the compacted tensors) of the common rows
    for b in range(B):
        common = np.intersect1d(g_rows[b], r_rows[b])
        gi.append(b * n_keep + np.searchsorted(g_rows[b], common))
        ri.append(b * n_keep + np.searchsorted(r_rows[b], common))
    gi, ri = np.concatenate(gi), np.concatenate(ri)
    flat_g = (np.arange(B)[:, None] * N + g_rows).reshape(-1)[gi]
    flat_r = (np.arange(B)[:, None] * N + r_rows).reshape(-1)[ri]
    rep = chain_report(W, dict(o=got["o"][flat_g], x1=got["x1"][gi], gu=got["gu"][gi], z=got["z"][gi], x_next=got["x_next"][gi]),
                       dict(o=ref["o"][flat_r], x1=ref["x1"][ri], gu=ref["gu"][ri], z=ref["z"][ri], x_next=ref["x_next"][ri]))
    rep["rows"] = len(gi)
    return rep, gi, ri


def chain_report(W, g, r):
    """Token-wise rest of the block, GPU tensors `g` against oracle tensors `r` (same rows): share of
    int4 codes that differ at the three quantizers (in front of O, gate/up, down), and whether every
    row whose quantized input (codes and scale) agrees is bit-exact behind the GEMM that follows."""
    rep = {}

    def codes(t):
        q, s_, _, _ = oracle.quantize_act(t)
        return q, s_

    def cmp(name, tg, tr):
        (qg, sg), (qr, sr) = codes(tg), codes(tr)
        rep[name] = float((qg != qr).mean())
        return np.all(qg == qr, axis=1) & (sg == sr)

    same2 = cmp("qa2", g["o"], r["o"])
    same3 = cmp("qa3", oracle.rmsnorm(g["x1"], W.gamma2, W.eps), oracle.rmsnorm(r["x1"], W.gamma2, W.eps))
    same4 = cmp("qa4", g["z"], r["z"])
    eq_rows = lambda a, b_: np.all(np.ascontiguousarray(a).view(np.uint16) == np.ascontiguousarray(b_).view(np.uint16), axis=1)
    x1_eq, gu_eq, xn_eq = eq_rows(g["x1"], r["x1"]), eq_rows(g["gu"], r["gu"]), eq_rows(g["x_next"], r["x_next"])
    # a GEMM is exact, so a row whose quantized input (codes and scale) and residual agree must agree bit for bit
    rep["x1_rows_checked"], rep["x1_ok"] = int(same2.sum()), bool(np.all(x1_eq[same2]))
    rep["gu_rows_checked"], rep["gu_ok"] = int(same3.sum()), bool(np.all(gu_eq[same3]))
    ok4 = same4 & x1_eq
    rep["xn_rows_checked"], rep["xn_ok"] = int(ok4.sum()), bool(np.all(xn_eq[ok4]))
    rep["rel_rms"] = dict(x1=rel_rms(g["x1"], r["x1"]), gu=rel_rms(g["gu"], r["gu"]), x_next=rel_rms(g["x_next"], r["x_next"]))
    return rep


def assert_chain_report(rep):
    for q in ("qa2", "qa3", "qa4"):
        assert rep[q] <= FLIP_BOUND[q], (q, rep[q])
    assert rep["x1_ok"] and rep["gu_ok"] and rep["xn_ok"], rep
    assert rep["rel_rms"]["x1"] < 1e-2 and rep["rel_rms"]["gu"] < 5e-2 and rep["rel_rms"]["x_next"] < 5e-2


def check_free_running(ref, got, shape, K, W):
    """Free-running chain (the GPU consumes its own floats) against the oracle.  fp16 tensors in front
    of the first re-quantization within 1e-2, scores within 1e-5 relative; kept sets equal except
    for tokens whose oracle score lies within that score tolerance of the cut (each printed); K/V
    codes of the common rows bit-exact.  Behind the attention output every tensor sits behind an
    int4 quantizer, where a one-ulp input difference can move a value by a whole quantization step:
    an element-wise fp16 bound cannot hold there (an earlier version of this test asserted it at the
    7B shape and failed on x1 and gu), so what is asserted instead is (a) the share of flipped int4
    codes at each quantizer stays under a stated bound and (b) every row whose quantized input did
    not flip is bit-exact behind the following GEMM.  The relative rms is reported as a secondary
    figure."""
    B, Nv = shape.B, shape.Nv
    k = min(K, Nv)
    n_keep = shape.N - Nv + k
    assert np.array_equal(np.ascontiguousarray(got["qkv"]).view(np.uint16), ref["qkv"].view(np.uint16))
    assert close_f16(got["o"], ref["o"])
    if Nv:
        assert close_f32(got["score"], ref["score"]), np.abs(got["score"] - ref["score"]).max()
    # index sets: equal, except swaps among tokens whose oracle scores are within the score tolerance of the cut
    for b in range(B):
        a, r = set(got["keep_idx"][b, :k].tolist()), set(ref["keep_idx"][b].tolist())
        if a != r:
            sc = ref["score"][b].astype(np.float64)
            cut = np.sort(sc)[::-1][k - 1]
            tol = 2e-5 * max(abs(cut), float(np.sqrt((sc ** 2).mean())))      # 1e-5 relative on either side
            for i in sorted(a ^ r):
                print(f"kept-set exception: sequence {b} token {i} score {sc[i]:.9g} cut {cut:.9g} gap {abs(sc[i] - cut):.3g}")
                assert abs(sc[i] - cut) <= tol, (b, i, sc[i], cut)
    if n_keep == 0:
        return None
    rep, gi, ri = free_running_report(ref, got, shape, K, W)
    print("free-running report:", rep)
    assert rep["rows"] >= B * (n_keep - 2 * 4)           # at most a few tokens swapped at the cut
    # K/V codes come from the bit-exact qkv: no float chain before them
    assert np.array_equal(got["cache_kc"][gi], ref["cache_kc"][ri]) and np.array_equal(got["cache_vc"][gi], ref["cache_vc"][ri])
    assert np.array_equal(got["pos_next"][gi], ref["pos_next"][ri])
    assert_chain_report(rep)
    assert rep["x1_rows_checked"] > 0
    return rep


def rel_rms(a, b):
    a = a.astype(np.float64)
    b = b.astype(np.float64)
    return float(np.sqrt(((a - b) ** 2).mean()) / max(np.sqrt((b ** 2).mean()), 1e-30))


def test_layer_small_free_running(qb):
    shape = wl.CONFIGS[0]
    W, L, cos, sin = build_layer(shape, 0)
    x, pos = wl.hidden_state(shape, 0), wl.positions(shape)
    for K in (19, 20):
        ref = oracle.prefill_layer(W, x, pos, 1, shape.N, 0, shape.Nv, K, cos, sin)
        got = run_gpu(qb, L, shape, x, pos, K)
        check_free_running(ref, got, shape, K, W)


def test_layer_7b_shape_full_size(qb):
    """The single 7B-shaped layer at its full size (640 tokens, keep 173), teacher-forced bit-exact and
    free-running within tolerance; the oracle needs a few tens of seconds on 8+ cores."""
    shape = wl.CONFIGS[1]
    W, L, cos, sin = build_layer(shape, 0)
    x, pos = wl.hidden_state(shape, 0), wl.positions(shape)
    K = wl.schedule_for(shape)[0]
    assert K == 173
    ref = oracle.prefill_layer(W, x, pos, 1, shape.N, 0, shape.Nv, K, cos, sin, prune_mid=True)
    got = run_gpu(qb, L, shape, x, pos, K, dict(o=ref["o"], z=ref["z"], cm_inter=ref["cm_inter"],
                                                cm_intra=ref["cm_intra"]))
    assert_teacher_forced_exact(ref, got, shape, K)
    free = run_gpu(qb, L, shape, x, pos, K)
    check_free_running(ref, free, shape, K, W)


def test_layer_errors(qb):
    from paper_2604_17320_amd.model import KVCache4
    shape = wl.CONFIGS[0]
    W, L, cos, sin = build_layer(shape, 1)
    x, pos = dev(wl.hidden_state(shape, 0)), dev(wl.positions(shape))
    x_out = torch.empty_like(x)
    pos_out = torch.empty_like(pos)
    ws = torch.empty(L.workspace_bytes(1, shape.N), dtype=torch.uint8, device="cuda")
    p = qb.quota_score_params_default()
    small = KVCache4(1, 10, shape.H, shape.dh)
    st = qb.State(1, shape.N, 0, shape.Nv, x.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    with pytest.raises(qb.QuotaError) as e:
        qb.quota_prefill_layer(L.desc, st, 19, p, small.desc, None, ws)
    assert e.value.code == qb.ERR_CAPACITY and small.len == 0 and st.N == shape.N
    st_bad = qb.State(1, shape.N, 70, shape.Nv, x.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    ok = KVCache4(1, 80, shape.H, shape.dh)
    with pytest.raises(qb.QuotaError) as e:
        qb.quota_prefill_layer(L.desc, st_bad, 19, p, ok.desc, None, ws)
    assert e.value.code == qb.ERR_INVALID_ARG


def test_layer_without_taps_equals_layer_with_taps(qb):
    """The benchmark runs the layer with no dump taps (the QKV projection then keeps no plain copy of
    its output); the result must be the same bits as the tapped run the parity tests check."""
    from paper_2604_17320_amd.model import KVCache4
    shape = wl.CONFIGS[0]
    W, L, cos, sin = build_layer(shape, 2)
    x, pos = wl.hidden_state(shape, 2), wl.positions(shape)
    K = 19
    tapped = run_gpu(qb, L, shape, x, pos, K)
    n_keep = shape.N - shape.Nv + K
    cache = KVCache4(1, n_keep, shape.H, shape.dh)
    x_out = torch.zeros((n_keep, shape.d), dtype=torch.float16, device="cuda")
    pos_out = torch.zeros((n_keep,), dtype=torch.int32, device="cuda")
    ws = torch.empty(L.workspace_bytes(1, shape.N), dtype=torch.uint8, device="cuda")
    xd, pd = dev(x), dev(pos)
    st = qb.State(1, shape.N, 0, shape.Nv, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, None, ws)
    assert np.array_equal(host(x_out).view(np.uint16), tapped["x_next"][:n_keep].view(np.uint16))
    assert np.array_equal(host(pos_out), tapped["pos_next"][:n_keep])
    assert np.array_equal(unpack4(host(cache.k_codes)[0, :n_keep]), tapped["cache_kc"])
    assert np.array_equal(host(cache.v_scales)[0, :n_keep].view(np.uint16), tapped["cache_vs"].view(np.uint16))


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
def test_layer_every_tile_with_fused_qkv_epilogue(qb, tile, pinned_gemm):
    """The QKV projection with its fused RoPE / KV-quantizer epilogue on each tile that carries it
    (and every other GEMM of the layer on the same tile), teacher-forced bit-exact."""
    pinned_gemm(tile)
    base = wl.CONFIGS[0]
    shape = wl.Shape("tile", d=base.d, H=base.H, F=base.F, layers=1, B=2, Nv=base.Nv, Nt=21,
                     n_outlier=base.n_outlier, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 3, gamma_random=True)
    x, pos = wl.hidden_state(shape, 3), wl.positions(shape)
    K = 19
    ref = oracle.prefill_layer(W, x, pos, shape.B, shape.N, 0, shape.Nv, K, cos, sin, prune_mid=True)
    got = run_gpu(qb, L, shape, x, pos, K, dict(o=ref["o"], z=ref["z"], cm_inter=ref["cm_inter"],
                                                cm_intra=ref["cm_intra"]))
    assert_teacher_forced_exact(ref, got, shape, K)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("Nv,Nt,K", [(500, 13, 499), (560, 17, 494)], ids=["513_to_512", "577_to_511"])
def test_layer_start_values_from_the_quantizer(qb, tile, Nv, Nt, K, pinned_gemm):
    """From 512 rows on the quantizers write the group sums' start values and the tiles read them: rows that end inside
    a tile, a last group of 96 channels, and a layer that falls below the line by pruning; teacher-forced bit-exact."""
    pinned_gemm(tile)
    base = wl.CONFIGS[0]
    shape = wl.Shape("starts", d=base.d, H=base.H, F=1376, layers=1, B=1, Nv=Nv, Nt=Nt, n_outlier=base.n_outlier, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 6, gamma_random=True)
    x, pos = wl.hidden_state(shape, 6), wl.positions(shape)
    ref = oracle.prefill_layer(W, x, pos, 1, shape.N, 0, Nv, K, cos, sin, prune_mid=True)
    got = run_gpu(qb, L, shape, x, pos, K, dict(o=ref["o"], z=ref["z"], cm_inter=ref["cm_inter"], cm_intra=ref["cm_intra"]))
    assert_teacher_forced_exact(ref, got, shape, K)


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3, 4])
@pytest.mark.parametrize("F,Nt,K", [(1376, 9, 8), (1376, 21, 19), (96, 30, 500), (2080, 30, 500)])
def test_layer_silu_product_in_the_gate_up_projection(qb, tile, F, Nt, K, pinned_gemm):
    """Without taps the gate/up projection makes SiLU(gate) * up itself: the bits of the run whose taps keep the two
    kernels apart, for channels that end inside a tile, 17 rows, ragged ones and start values (530 rows)."""
    from paper_2604_17320_amd.model import KVCache4
    pinned_gemm(tile)
    base = wl.CONFIGS[0]
    shape = wl.Shape("silu", d=base.d, H=base.H, F=F, layers=1, B=1, Nv=500, Nt=Nt, n_outlier=base.n_outlier, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 7)
    x, pos = wl.hidden_state(shape, 7), wl.positions(shape)
    tapped = run_gpu(qb, L, shape, x, pos, K)
    n_keep = shape.N - 500 + K
    cache = KVCache4(1, n_keep, shape.H, shape.dh)
    x_out = torch.zeros((n_keep, shape.d), dtype=torch.float16, device="cuda")
    pos_out = torch.zeros((n_keep,), dtype=torch.int32, device="cuda")
    ws = torch.empty(L.workspace_bytes(1, shape.N), dtype=torch.uint8, device="cuda")
    xd, pd = dev(x), dev(pos)
    st = qb.State(1, shape.N, 0, 500, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, None, ws)
    assert np.array_equal(host(x_out).view(np.uint16), tapped["x_next"][:n_keep].view(np.uint16))


@pytest.mark.parametrize("d,dh,F,N", [(2048, 128, 2048, 480), (2048, 128, 2048, 641), (1024, 128, 1376, 1000), (1024, 64, 1376, 100),
                                      (1024, 64, 96, 33), (1152, 128, 11008, 132), (1152, 128, 11008, 170), (4096, 128, 1376, 331),
                                      (640, 128, 18944, 68), (640, 128, 18944, 99)])
def test_layer_tiles_in_long_stages(qb, d, dh, F, N, pinned_gemm):
    """The tiles of the choice, in stages of four groups, with and without start values, and 32 x 64 in stages of eight, which
    only the choice takes (100 and 33 rows), as it does 96 x 128 (gate/up of 22016 and 37888 columns, QKV of 12288), over whole and ragged numbers of groups: the bits of the pinned 128 x 128 tile."""
    from paper_2604_17320_amd.model import KVCache4
    shape = wl.Shape("stages", d=d, H=d // dh, F=F, layers=1, B=1, Nv=N - 8, Nt=8, n_outlier=4, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 9)
    x, pos = wl.hidden_state(shape, 9), wl.positions(shape)
    K = N - 11
    got = []
    for tile in (0, -1):
        pinned_gemm(tile)
        tapped = run_gpu(qb, L, shape, x, pos, K)
        cache = KVCache4(1, K + 8, shape.H, dh)
        x_out, pos_out = torch.zeros((K + 8, d), dtype=torch.float16, device="cuda"), torch.zeros((K + 8,), dtype=torch.int32, device="cuda")
        ws = torch.empty(L.workspace_bytes(1, N), dtype=torch.uint8, device="cuda")
        xd, pd = dev(x), dev(pos)
        st = qb.State(1, N, 0, N - 8, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
        qb.quota_profile_begin(64)
        qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, None, ws)
        ran = {n: s["launches"] for n, s in qb.quota_profile_collect().items() if n.startswith("w4a4")}
        assert tile >= 0 or ran.get("w4a4_gemm_96x128", 0) == (1 if F > 10000 or d == 4096 else 0), ran
        got.append([tapped[k] for k in ("qkv", "q_rot", "x1", "gu", "x_next")] + [host(x_out)])
    for a, b in zip(*got):
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16))


@pytest.mark.parametrize("rows", [449, 480, 481, 511])
def test_layer_96_row_tile_adds_the_residual(qb, rows, pinned_gemm):
    """O and down on the tile of 96 rows, whose three rounds of the epilogue ask for all residual rows at once, for rows that end in the first
    round of a tile, with it, and one behind it: the bits of the pinned 128 x 128 tile."""
    from paper_2604_17320_amd.model import KVCache4, PackedLinear, PrefillLayer
    d, H, F, N, Nv = 8320, 65, 1024, 520, 512              # (520 rows of QKV are on another tile)
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    def linear(n, k):
        codes = torch.randint(-8, 8, (n, k), generator=g, device="cuda", dtype=torch.int8)
        scales = (torch.rand((n, k // 128), generator=g, device="cuda") * 0.002 + 0.001).to(torch.float16)
        return PackedLinear.from_codes(codes, scales)
    cos, sin = (dev(t) for t in wl.rope_tables(128, N))
    ones = torch.ones(d, device="cuda")
    L = PrefillLayer(H, 128, F, linear(d + 2 * 128, d), linear(d, d), linear(2 * F, d), linear(d, F), ones, ones, 1e-5, cos, sin, 1)
    x = torch.randn((N, d), generator=g, device="cuda").to(torch.float16)
    pos = torch.arange(N, dtype=torch.int32, device="cuda")
    outs = []
    for tile in (0, -1):
        pinned_gemm(tile)
        cache = KVCache4(1, rows, 1, 128)
        x_out, pos_out = torch.full((rows, d), float("nan"), dtype=torch.float16, device="cuda"), torch.zeros(rows, dtype=torch.int32, device="cuda")
        ws = torch.full((L.workspace_bytes(1, N),), 0xFF, dtype=torch.uint8, device="cuda")
        st = qb.State(1, N, 0, Nv, x.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
        qb.quota_profile_begin(64)
        qb.quota_prefill_layer(L.desc, st, rows - (N - Nv), qb.quota_score_params_default(), cache.desc, None, ws)
        ran = {n: s["launches"] for n, s in qb.quota_profile_collect().items() if n.startswith("w4a4")}
        assert ran.get("w4a4_gemm_96x128", 0) == (0 if tile == 0 else 2), ran
        outs.append(host(x_out))
    assert np.isfinite(outs[0].astype(np.float32)).all()
    assert np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))


# A layer that picks its kept rows (33 to 511 of at most 1024): the fewest, sequences with text on both sides, a single kept token, rows of two and of four chunks a
# thread, the most rows in and kept, each pinned tile; and beside each limit, where it gathers them.
@pytest.mark.parametrize("tile,H,Hkv,dh,B,N,vb,Nv,K", [(-1, 8, 8, 64, 1, 80, 0, 64, 17), (-1, 8, 8, 64, 1, 80, 0, 64, 16), (-1, 8, 4, 64, 3, 101, 14, 70, 1),
                                                       (-1, 40, 8, 128, 1, 333, 30, 290, 157), (-1, 8, 8, 64, 1, 1024, 1, 1020, 507),
                                                       (-1, 8, 8, 64, 1, 1024, 1, 1020, 508), (-1, 8, 8, 64, 1, 1025, 0, 1024, 300),
                                                       (-1, 10, 2, 128, 2, 512, 5, 500, 200), (0, 8, 8, 64, 2, 200, 7, 150, 60), (1, 8, 8, 64, 2, 200, 7, 150, 60),
                                                       (2, 8, 8, 64, 2, 200, 7, 150, 60), (3, 8, 8, 64, 2, 200, 7, 150, 60), (4, 8, 8, 64, 2, 200, 7, 150, 60)])
def test_layer_that_picks_its_rows(qb, tile, H, Hkv, dh, B, N, vb, Nv, K, pinned_gemm):
    """Hidden state, positions, kept rows and cache have the bits of the layer whose output projection, with weight scales between two dwords, takes gathered
    rows; the launches say which of the two ran."""
    from paper_2604_17320_amd.model import KVCache4, PackedLinear, PrefillLayer, make_taps
    d, F, n_keep = H * dh, 640, N - Nv + K
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K)
    def linear(n, k):
        codes = torch.randint(-8, 8, (n, k), generator=g, device="cuda", dtype=torch.int8)
        scales = (torch.rand((n, (k + 127) // 128), generator=g, device="cuda") * 0.002 + 0.001).to(torch.float16)
        return PackedLinear.from_codes(codes, scales)
    cos, sin = (dev(t) for t in wl.rope_tables(dh, N))
    ones = torch.ones(d, device="cuda")
    L = PrefillLayer(H, dh, F, linear(d + 2 * Hkv * dh, d), linear(d, d), linear(2 * F, d), linear(d, F), ones, ones, 1e-5, cos, sin, Hkv)
    x = torch.randn((B * N, d), generator=g, device="cuda").to(torch.float16)
    pos = torch.arange(N, dtype=torch.int32, device="cuda").repeat(B) + 3
    odd = torch.cat([L.o.scales.new_zeros(1), L.o.scales.flatten()])
    even = L.desc.o.scales
    outs = []
    for scales in (odd[1:].data_ptr(), even):
        L.desc.o.scales = scales
        pinned_gemm(tile)
        cache = KVCache4(B, n_keep + 3, Hkv, dh)
        for t in (cache.k_codes, cache.v_codes, cache.k_scales, cache.v_scales):
            t.zero_()
        cache.desc.len = 2
        x_out = torch.full((B * n_keep, d), float("nan"), dtype=torch.float16, device="cuda")
        pos_out, rows = (torch.full((B * n_keep,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ws = torch.full((L.workspace_bytes(B, N),), 0xFF, dtype=torch.uint8, device="cuda")
        st = qb.State(B, N, vb, Nv, x.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
        qb.quota_profile_begin(64)
        qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, make_taps(rows=rows), ws)
        gathers = qb.quota_profile_collect().get("compact_rows", {}).get("launches", 0)
        assert gathers == (0 if scales == even and 32 < B * n_keep < 512 and B * N <= 1024 and Nv <= 1024 else 1)
        assert (st.N, st.Nv, cache.len) == (n_keep, K, n_keep + 2)
        outs.append([host(t) for t in (x_out, pos_out, rows, cache.k_codes, cache.v_codes, cache.k_scales, cache.v_scales)])
    assert np.isfinite(outs[0][0].astype(np.float32)).all()
    for a, b in zip(*outs):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))


@pytest.mark.parametrize("H,Hkv,dh,B,N,Nv,K", [(8, 8, 64, 1, 80, 64, 17), (16, 4, 128, 3, 101, 70, 20)])
def test_profile_of_a_layer_that_picks_its_rows(qb, H, Hkv, dh, B, N, Nv, K):
    """The score launch counts the attention rows that are quantized beside it, the second RMSNorm's the kept K/V, positions and numbers that it copies."""
    from paper_2604_17320_amd.model import KVCache4, PackedLinear, PrefillLayer
    d, dkv, F, n_keep = H * dh, Hkv * dh, 640, N - Nv + K
    def linear(n, k):
        return PackedLinear.from_codes(torch.ones((n, k), device="cuda", dtype=torch.int8), torch.full((n, (k + 127) // 128), 0.001, device="cuda").to(torch.float16))
    cos, sin = (dev(t) for t in wl.rope_tables(dh, N))
    ones = torch.ones(d, device="cuda")
    L = PrefillLayer(H, dh, F, linear(d + 2 * dkv, d), linear(d, d), linear(2 * F, d), linear(d, F), ones, ones, 1e-5, cos, sin, Hkv)
    x = torch.randn((B * N, d), generator=torch.Generator(device="cuda").manual_seed(N), device="cuda").to(torch.float16)
    pos = torch.arange(N, dtype=torch.int32, device="cuda").repeat(B)
    x_out, pos_out = torch.empty((B * n_keep, d), dtype=torch.float16, device="cuda"), torch.empty(B * n_keep, dtype=torch.int32, device="cuda")
    ws = torch.empty(L.workspace_bytes(B, N), dtype=torch.uint8, device="cuda")
    st = qb.State(B, N, 0, Nv, x.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    cache = KVCache4(B, n_keep, Hkv, dh)
    qb.quota_profile_begin(64)
    qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, None, ws)
    ran = qb.quota_profile_collect()
    assert "compact_rows" not in ran and ran["rmsnorm_quantize_act"]["launches"] == 2
    rows = lambda M: 2.5 * M * d + 4 * M                  # fp16 in, half a byte and a token scale out
    kept = 2 * (dkv // 2) + 2 * 2 * (dkv // 64)           # codes and fp16 scales of K and V of a row
    assert ran["score_tokens"]["bytes"] == 20 * B * Nv + 4 * B * K + rows(B * N)
    assert ran["rmsnorm_quantize_act"]["bytes"] == rows(B * N) + rows(B * n_keep) + 2 * 4 * d + B * n_keep * (2 * kept + 2 * 4 + 4)


def test_layer_with_weight_scales_at_an_odd_halfword(qb):
    """Weight scales that start between two dwords: a prefill layer and its decode-sized remainder give the bits of the
    aligned layer (the fused QKV epilogue and the tiles step aside)."""
    from paper_2604_17320_amd.model import PrefillLayer
    base = wl.CONFIGS[0]
    shape = wl.Shape("odd", d=base.d, H=base.H, F=base.F, layers=1, B=2, Nv=base.Nv, Nt=21, n_outlier=base.n_outlier,
                     vis_begin=0)
    W, L, cos, sin = build_layer(shape, 4, gamma_random=True)
    x, pos = wl.hidden_state(shape, 4), wl.positions(shape)
    want = run_gpu(qb, L, shape, x, pos, 19)
    keep = []
    for name in ("qkv", "o", "gu", "down"):
        lin = getattr(L, name)
        keep.append(torch.cat([lin.scales.new_zeros(1), lin.scales]))
        lin.desc.scales = keep[-1][1:].data_ptr()
        assert lin.desc.scales % 4 == 2
    odd = PrefillLayer(L.H, L.dh, L.F, L.qkv, L.o, L.gu, L.down, L.gamma1, L.gamma2, 1e-5, L.cosT, L.sinT)
    got = run_gpu(qb, odd, shape, x, pos, 19)
    for name in want:
        assert np.array_equal(want[name], got[name]), name


@pytest.mark.parametrize("off", [1, 4, 8, 15])
def test_layer_workspace_anywhere(qb, off):
    """A workspace that starts `off` bytes behind a multiple of 16: the bits of one that starts there, in a pruned prefill
    layer and in a decode step whose cached rows are split over workgroups, and not a byte touched outside its size."""
    from paper_2604_17320_amd.model import KVCache4
    base = wl.CONFIGS[0]
    shape = wl.Shape("ws", d=base.d, H=base.H, F=base.F, layers=1, B=2, Nv=base.Nv, Nt=21, n_outlier=base.n_outlier, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 3)
    B, N, K, rows = shape.B, shape.N, 30, 1700
    n = N - shape.Nv + K
    xd, pd = dev(wl.hidden_state(shape, 3)), dev(wl.positions(shape))
    long_cache = [torch.from_numpy(wl.rng(3, "ws", i).integers(0, 256, s, dtype=np.uint8)).cuda()
                  for i, s in enumerate([(B, rows + 1, shape.d // 2)] * 2)]
    outs = []
    for o in (0, off):
        def room(nbytes):
            t = torch.full((o + nbytes + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            rooms.append((t, nbytes))
            return t[o: o + nbytes]
        rooms = []
        cache = KVCache4(B, n, shape.H, shape.dh)
        x_out = torch.zeros((B * n, shape.d), dtype=torch.float16, device="cuda")
        pos_out = torch.zeros((B * n,), dtype=torch.int32, device="cuda")
        st = qb.State(B, N, 0, shape.Nv, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
        qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, None, room(L.workspace_bytes(B, N)))
        grown = KVCache4(B, rows + 1, shape.H, shape.dh)
        grown.k_codes.copy_(long_cache[0])
        grown.v_codes.copy_(long_cache[1])
        grown.k_scales.fill_(0.25)
        grown.v_scales.fill_(0.25)
        grown.desc.len = rows
        y = torch.zeros((B, shape.d), dtype=torch.float16, device="cuda")
        L.decode(x_out[:B], pos_out[:B], grown, y, room(L.decode_workspace_bytes(B)))
        for t, nbytes in rooms:
            assert bool((t[:o] == 0xA5).all()) and bool((t[o + nbytes:] == 0xA5).all())
        outs.append([t.view(torch.uint8) for t in (x_out, cache.k_codes, cache.k_scales, cache.v_codes, cache.v_scales, y)])
    assert bool(torch.isfinite(outs[0][-1].view(torch.float16)).all())
    assert all(torch.equal(a, b) for a, b in zip(*outs))


def test_layer_with_weights_fetched_ahead(qb):
    """One sequence, whose attention and cue pass leave CUs to the fetch of the later projections' weights, and four of the same, whose
    launches leave none: the same bits in each, with 64-channel heads and weight scales that start between two 16-byte pieces."""
    shape = wl.Shape("ahead", d=1024, H=16, F=2816, layers=1, B=1, Nv=500, Nt=20, n_outlier=10, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 11)
    keep = []
    for name in ("qkv", "o", "gu", "down"):
        lin = getattr(L, name)
        keep.append(torch.cat([lin.scales.new_zeros(2), lin.scales]))
        lin.desc.scales = keep[-1][2:].data_ptr()
        assert lin.desc.scales % 16 == 4
    from paper_2604_17320_amd.model import PrefillLayer
    L = PrefillLayer(L.H, L.dh, L.F, L.qkv, L.o, L.gu, L.down, L.gamma1, L.gamma2, 1e-5, L.cosT, L.sinT)
    four = wl.Shape("four", **{**{k: getattr(shape, k) for k in ("d", "H", "F", "layers", "Nv", "Nt", "n_outlier", "vis_begin")}, "B": 4})
    x, pos = wl.hidden_state(shape, 11), wl.positions(shape)
    one = run_gpu(qb, L, shape, x, pos, 100)
    many = run_gpu(qb, L, four, np.tile(x, (4, 1)), np.tile(pos, 4), 100)
    for name in ("qkv", "o", "cm_inter", "cm_intra", "score", "keep_idx", "x1", "z", "x_next", "cache_kc", "cache_vs"):
        for part in np.split(many[name], 4):
            assert part.tobytes() == one[name].tobytes(), name


def test_long_top_k_beside_the_fetch(qb):
    """More than 3072 visual tokens with eight heads: attention and cues fill the chip, score and top-k run beside the fetch."""
    shape = wl.Shape("long", d=512, H=8, F=5632, layers=1, B=1, Nv=3100, Nt=100, n_outlier=4, vis_begin=0)
    W, L, cos, sin = build_layer(shape, 12)
    got = run_gpu(qb, L, shape, wl.hidden_state(shape, 12), wl.positions(shape), 77)
    score = oracle.score(got["sumsq"], got["ressq"], got["cm_inter"], got["cm_intra"])
    assert np.array_equal(got["score"].view(np.uint32), score.view(np.uint32))
    assert np.array_equal(got["keep_idx"], oracle.topk(score, 77))


@pytest.mark.parametrize("Nv", [1, 2, 63, 64, 65, 256, 257, 576, 1023, 1024, 1025])
def test_selection_of_tied_tokens(qb, Nv):
    """Visual tokens that are copies of nine, under flat cues: most scores are tied, and the threshold falls among them.  Around the sizes where
    a wave's registers of keys and the kernel change."""
    shape = wl.Shape("ties", d=512, H=8, F=1376, layers=1, B=2, Nv=Nv, Nt=9, n_outlier=4, vis_begin=3)
    W, L, cos, sin = build_layer(shape, 13)
    r = wl.rng(13, "ties", Nv)
    x = wl.hidden_state(shape, 13).reshape(2, shape.N, shape.d).copy()
    x[:, 3:3 + Nv] = x[:, 3:4 + min(Nv - 1, 8)][:, r.integers(0, min(Nv, 9), Nv)]
    flat = np.full((2, Nv), 0.5, np.float32)
    for K in sorted({1, Nv // 3, Nv - 1, Nv} - {0}):
        got = run_gpu(qb, L, shape, x.reshape(-1, shape.d), wl.positions(shape), K, dict(cm_inter=flat, cm_intra=flat))
        score = oracle.score(got["sumsq"], got["ressq"], flat, flat)
        assert np.array_equal(got["score"].view(np.uint32), score.view(np.uint32)), K
        assert np.array_equal(got["keep_idx"], oracle.topk(score, K)), K


@pytest.mark.parametrize("H,Nv", [(8, 1), (8, 257), (8, 1024), (8, 1025), (10, 255), (20, 512), (20, 513), (40, 256)])
def test_head_means_in_the_score_kernel(qb, H, Nv):
    """Few masses: their head means are the score kernel's; with cues handed in they are a launch of their own.  Both have the same bits, and so
    has what follows from them.  Around the sizes where the one or the other is chosen, uneven quarters of the heads."""
    shape = wl.Shape("means", d=64 * H, H=H, F=256, layers=1, B=2, Nv=Nv, Nt=5, n_outlier=4, vis_begin=2)
    W, L, cos, sin = build_layer(shape, 21)
    x, pos, K = wl.hidden_state(shape, 21), wl.positions(shape), max(1, Nv // 3)
    got = run_gpu(qb, L, shape, x, pos, K)
    apart = run_gpu(qb, L, shape, x, pos, K, dict(cm_inter=got["cm_inter"], cm_intra=got["cm_intra"]))
    for name in ("cm_inter", "cm_intra", "score", "keep_idx", "x_next"):
        assert np.array_equal(got[name].view(np.uint8), apart[name].view(np.uint8)), name
    score = oracle.score(got["sumsq"], got["ressq"], got["cm_inter"], got["cm_intra"])
    assert np.array_equal(got["score"].view(np.uint32), score.view(np.uint32))
