"""GPU parity with grouped-query attention (fewer K/V heads than query heads, as in the paper's
second model family): the attention entry points on their own, then a whole layer (prefill,
teacher-forced bit-exact, the narrower 4-bit cache) and decode steps over that cache."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17320_amd import workloads as wl
from test_gpu_ops import _act, _pack4, close_f16, dev, host, unpack4
from test_gpu_layer import assert_chain_report, chain_report
from test_gpu_decode import eq16, fill_cache

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    assert torch.cuda.is_available()
    from paper_2604_17320_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("B,N,H,Hkv,dh,vb,Nv", [(2, 150, 6, 2, 64, 3, 100), (1, 300, 8, 2, 128, 0, 260),
                                                 (1, 70, 4, 1, 128, 0, 50)])
def test_attention_prefill_gqa(qb, B, N, H, Hkv, dh, vb, Nv):
    q = _act(B * N, H * dh, 91, 1.0)
    _, _, khat = oracle.kv_quant(_act(B * N, Hkv * dh, 92, 1.0))
    _, _, vhat = oracle.kv_quant(_act(B * N, Hkv * dh, 93, 1.0))
    o_ref, ci_ref, cv_ref = oracle.attention(q, khat, vhat, B, N, H, dh, vb, Nv, Hkv=Hkv)
    o = torch.empty((B * N, H * dh), dtype=torch.float16, device="cuda")
    ci, cv = (torch.zeros((B, Nv), dtype=torch.float32, device="cuda") for _ in range(2))
    ws = torch.empty(qb.quota_attention_workspace_bytes(B, N, H, dh), dtype=torch.uint8, device="cuda")
    qb.quota_attention_prefill_gqa(dev(q), dev(khat), dev(vhat), B, N, H, Hkv, dh, vb, Nv, o, ci, cv, ws)
    assert close_f16(host(o), o_ref)
    assert np.allclose(host(ci), ci_ref, rtol=2e-5, atol=1e-7) and np.allclose(host(cv), cv_ref, rtol=2e-5, atol=1e-7)


def test_attention_decode_gqa(qb):
    from paper_2604_17320_amd.model import KVCache4
    B, L, Hq, Hkv, dh = 3, 210, 8, 2, 128
    r = wl.rng(94, "gqa-dec")
    kc, ks, _ = oracle.kv_quant((r.standard_normal((B * L, Hkv * dh)) * 1.5).astype(np.float16))
    vc, vs, _ = oracle.kv_quant(r.standard_normal((B * L, Hkv * dh)).astype(np.float16))
    sh = lambda a: a.reshape(B, L, -1)
    c = dict(kc=sh(kc), ks=sh(ks), vc=sh(vc), vs=sh(vs))
    q = r.standard_normal((B, Hq * dh)).astype(np.float16)
    ref = oracle.decode_attention(q, c["kc"], c["ks"], c["vc"], c["vs"], Hq, dh, Hkv)
    cache = KVCache4(B, L + 2, Hkv, dh)
    fill_cache(cache, c, L)
    o = torch.zeros((B, Hq * dh), dtype=torch.float16, device="cuda")
    qb.quota_attention_decode_gqa(dev(q), Hq, cache.desc, o)
    assert close_f16(host(o), ref)
    with pytest.raises(qb.QuotaError) as e:
        qb.quota_attention_decode_gqa(dev(q), 7, cache.desc, o)       # 7 query heads over 2 K/V heads
    assert e.value.code == qb.ERR_SHAPE


@pytest.mark.parametrize("B,L,Hq,Hkv,dh", [
    (2, 700, 28, 4, 128),      # 7 query heads per K/V head: the last workgroup of a head serves one query head
    (3, 513, 6, 3, 64),        # head_dim 64, one row past a 512-row tile, a grid that is no multiple of 8
    (1, 512, 4, 1, 128),       # exactly one tile, one K/V head
    (5, 1100, 10, 5, 128),     # three tiles of the running softmax
])
def test_attention_decode_gqa_shapes(qb, B, L, Hq, Hkv, dh):
    """Grouped heads through the decode attention's workgroup layout: one workgroup per (sequence,
    K/V head, pair of query heads), dealt to the XCDs in contiguous ranges."""
    from paper_2604_17320_amd.model import KVCache4
    r = wl.rng(95, "gqa-dec", B, L, Hq)
    kc, ks, _ = oracle.kv_quant((r.standard_normal((B * L, Hkv * dh)) * 1.5).astype(np.float16))
    vc, vs, _ = oracle.kv_quant(r.standard_normal((B * L, Hkv * dh)).astype(np.float16))
    sh = lambda a: a.reshape(B, L, -1)
    c = dict(kc=sh(kc), ks=sh(ks), vc=sh(vc), vs=sh(vs))
    q = r.standard_normal((B, Hq * dh)).astype(np.float16)
    ref = oracle.decode_attention(q, c["kc"], c["ks"], c["vc"], c["vs"], Hq, dh, Hkv)
    cache = KVCache4(B, L + 3, Hkv, dh)
    fill_cache(cache, c, L)
    o = torch.full((B, Hq * dh), float("nan"), dtype=torch.float16, device="cuda")     # every output must be written
    qb.quota_attention_decode_gqa(dev(q), Hq, cache.desc, o)
    assert close_f16(host(o), ref)


def build_gqa_layer(d, H, Hkv, dh, F, seed, n_pos):
    from paper_2604_17320_amd.model import PackedLinear, PrefillLayer
    r = wl.rng(seed, "gqa-layer")
    mk = lambda n, k: oracle.quantize_weights((r.standard_normal((n, k)) * 0.02).astype(np.float32))
    q = dict(qkv=mk(d + 2 * Hkv * dh, d), o=mk(d, d), gu=mk(2 * F, d), down=mk(d, F))
    g1 = r.uniform(0.7, 1.3, d).astype(np.float32)
    g2 = r.uniform(0.7, 1.3, d).astype(np.float32)
    W = oracle.LayerWeights(qkv=q["qkv"], o=q["o"], gu=q["gu"], down=q["down"], gamma1=g1, gamma2=g2, eps=1e-5,
                            H=H, dh=dh, F=F, Hkv=Hkv)
    cos, sin = wl.rope_tables(dh, n_pos)
    lin = {k: PackedLinear.from_codes(dev(c), dev(s)) for k, (c, s) in q.items()}
    L = PrefillLayer(H, dh, F, lin["qkv"], lin["o"], lin["gu"], lin["down"], dev(g1), dev(g2), 1e-5, dev(cos),
                     dev(sin), Hkv=Hkv)
    return W, L, cos, sin


@pytest.mark.parametrize("d,H,Hkv,dh,F,B,Nv,Nt,K", [(512, 8, 2, 64, 1376, 2, 64, 16, 19),
                                                    (1024, 8, 2, 128, 2048, 1, 200, 24, 60),
                                                    (256, 4, 1, 64, 160, 2, 40, 8, 11)])   # K/V width 64: unfused path
def test_layer_gqa_prefill_then_decode(qb, d, H, Hkv, dh, F, B, Nv, Nt, K):
    from paper_2604_17320_amd.model import KVCache4, make_taps
    N, dkv = Nv + Nt, Hkv * dh
    shape = wl.Shape("gqa", d=d, H=H, F=F, layers=1, B=B, Nv=Nv, Nt=Nt, n_outlier=4, vis_begin=0)
    W, L, cos, sin = build_gqa_layer(d, H, Hkv, dh, F, 7, N + 8)
    x, pos = wl.hidden_state(shape, 7), wl.positions(shape)
    ref = oracle.prefill_layer(W, x, pos, B, N, 0, Nv, K, cos, sin, prune_mid=True)
    n_keep = N - Nv + K
    t16 = lambda *shp: torch.zeros(shp, dtype=torch.float16, device="cuda")
    out = dict(qkv=t16(B * N, d + 2 * dkv), q_rot=t16(B * N, d), o=t16(B * N, d), x1=t16(B * n_keep, d),
               gu=t16(B * n_keep, 2 * F), score=torch.zeros((B, Nv), dtype=torch.float32, device="cuda"),
               keep_idx=torch.zeros((B, K), dtype=torch.int32, device="cuda"))
    inj = {k: dev(ref[k]) for k in ("o", "z", "cm_inter", "cm_intra")}
    taps = make_taps(**out, inject_o=inj["o"], inject_z=inj["z"], inject_cm_inter=inj["cm_inter"],
                     inject_cm_intra=inj["cm_intra"])
    cache = KVCache4(B, n_keep + 4, Hkv, dh)
    x_out, pos_out = t16(B * n_keep, d), torch.zeros((B * n_keep,), dtype=torch.int32, device="cuda")
    ws = torch.empty(L.workspace_bytes(B, N), dtype=torch.uint8, device="cuda")
    xd, pd = dev(x), dev(pos)
    st = qb.State(B, N, 0, Nv, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    qb.quota_prefill_layer(L.desc, st, K, qb.quota_score_params_default(), cache.desc, taps, ws)
    assert eq16(host(out["qkv"]), ref["qkv"]) and eq16(host(out["q_rot"]), ref["q"])
    assert np.array_equal(host(out["score"]), ref["score"]) and np.array_equal(host(out["keep_idx"]), ref["keep_idx"])
    assert cache.len == n_keep and cache.k_codes.shape[-1] == dkv // 2
    assert np.array_equal(unpack4(host(cache.k_codes)[:, :n_keep]).reshape(B * n_keep, dkv), ref["cache_kc"])
    assert np.array_equal(unpack4(host(cache.v_codes)[:, :n_keep]).reshape(B * n_keep, dkv), ref["cache_vc"])
    assert eq16(host(cache.k_scales)[:, :n_keep].reshape(B * n_keep, -1), ref["cache_ks"])
    assert eq16(host(out["x1"]), ref["x1"]) and eq16(host(out["gu"]), ref["gu"]) and eq16(host(x_out), ref["x_next"])
    assert close_f16(host(out["o"]), ref["o"])              # the library's own attention, dumped by the same run

    # decode over the pruned, narrower cache
    ocache = oracle.cache_from_prefill(ref, B)
    r = wl.rng(8, "gqa-dec-x")
    dws = torch.empty(L.decode_workspace_bytes(B), dtype=torch.uint8, device="cuda")
    for step in range(2):
        xn = r.standard_normal((B, d)).astype(np.float16)
        pn = np.full(B, N + step, np.int32)
        dref = oracle.decode_layer(W, xn, pn, ocache, cos, sin)
        dout = dict(q_rot=t16(B, d), o=t16(B, d), x1=t16(B, d))
        di = {k: dev(dref[k]) for k in ("o", "z")}
        y = t16(B, d)
        Lc = cache.len
        L.decode(dev(xn), dev(pn), cache, y, dws, make_taps(**dout, inject_o=di["o"], inject_z=di["z"]))
        assert cache.len == Lc + 1
        assert eq16(host(dout["q_rot"]), dref["q"]) and eq16(host(dout["x1"]), dref["x1"]) and eq16(host(y), dref["x_next"])
        assert np.array_equal(unpack4(host(cache.k_codes)[:, Lc]), dref["kc"])
        assert eq16(host(cache.v_scales)[:, Lc], dref["vs"])
        assert close_f16(host(dout["o"]), dref["o"])
        free = t16(B, d)
        fo = dict(o=t16(B, d), x1=t16(B, d), gu=t16(B, 2 * F), z=t16(B, F))
        cache.desc.len = Lc                                  # same step again, free-running
        L.decode(dev(xn), dev(pn), cache, free, dws, make_taps(**fo))
        rep = chain_report(W, dict({k_: host(v_) for k_, v_ in fo.items()}, x_next=host(free)), dref)
        print("gqa decode free-running report:", rep)
        assert_chain_report(rep)
        ocache = dref["cache"]


def test_layer_qwen25_vl_7b_shape(qb):
    """One layer at the shape of the paper's second model family (Qwen2.5-VL-7B language model:
    d = 3584, 28 query heads over 4 K/V heads of 128, SwiGLU FFN 18944 -- wider than the 16384 columns
    one workgroup row used to hold), 300 visual + 20 text tokens, budget 90 (30 %): prefill
    teacher-forced bit-exact incl. the narrow 4-bit cache; then the same layer as a layer outside the
    candidate set (supplementary: pruning at layers 8-12 only), which must keep every token."""
    from paper_2604_17320_amd.model import KVCache4, make_taps
    d, H, Hkv, dh, F, B, Nv, Nt, K = 3584, 28, 4, 128, 18944, 1, 300, 20, 90
    N, dkv = Nv + Nt, Hkv * dh
    W, L, cos, sin = build_gqa_layer(d, H, Hkv, dh, F, 21, N + 8)
    shape = wl.Shape("qwen", d=d, H=H, F=F, layers=1, B=B, Nv=Nv, Nt=Nt, n_outlier=36, vis_begin=0)
    x, pos = wl.hidden_state(shape, 21), wl.positions(shape)
    t16 = lambda *shp: torch.zeros(shp, dtype=torch.float16, device="cuda")
    for K_l, K_or in ((K, K), (qb.KEEP_ALL, Nv)):
        print("qwen-shaped layer, K_l =", K_l, flush=True)
        ref = oracle.prefill_layer(W, x, pos, B, N, 0, Nv, K_or, cos, sin, prune_mid=True)
        n_keep = N - Nv + K_or
        out = dict(qkv=t16(B * N, d + 2 * dkv), q_rot=t16(B * N, d), o=t16(B * N, d), x1=t16(B * n_keep, d),
                   gu=t16(B * n_keep, 2 * F), keep_idx=torch.full((B, K_or), -1, dtype=torch.int32, device="cuda"))
        inj = {k: dev(ref[k]) for k in ("o", "z", "cm_inter", "cm_intra")}
        taps = make_taps(**out, inject_o=inj["o"], inject_z=inj["z"], inject_cm_inter=inj["cm_inter"],
                         inject_cm_intra=inj["cm_intra"])
        cache = KVCache4(B, n_keep + 2, Hkv, dh)
        x_out, pos_out = t16(B * n_keep, d), torch.zeros((B * n_keep,), dtype=torch.int32, device="cuda")
        ws = torch.empty(L.workspace_bytes(B, N), dtype=torch.uint8, device="cuda")
        xd, pd = dev(x), dev(pos)
        st = qb.State(B, N, 0, Nv, xd.data_ptr(), pd.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
        qb.quota_prefill_layer(L.desc, st, K_l, qb.quota_score_params_default(), cache.desc, taps, ws)
        assert (st.N, st.Nv, cache.len) == (n_keep, K_or, n_keep)
        assert eq16(host(out["qkv"]), ref["qkv"]) and eq16(host(out["q_rot"]), ref["q"])
        if K_l == qb.KEEP_ALL:
            assert np.all(host(out["keep_idx"]) == -1)                     # no selection ran
        else:
            assert np.array_equal(host(out["keep_idx"]), ref["keep_idx"])
        assert np.array_equal(host(pos_out), ref["pos_next"])
        assert np.array_equal(unpack4(host(cache.k_codes)[:, :n_keep]).reshape(B * n_keep, dkv), ref["cache_kc"])
        assert np.array_equal(unpack4(host(cache.v_codes)[:, :n_keep]).reshape(B * n_keep, dkv), ref["cache_vc"])
        assert eq16(host(cache.v_scales)[:, :n_keep].reshape(B * n_keep, -1), ref["cache_vs"])
        assert eq16(host(out["x1"]), ref["x1"]) and eq16(host(out["gu"]), ref["gu"]) and eq16(host(x_out), ref["x_next"])
        assert close_f16(host(out["o"]), ref["o"])


@pytest.mark.parametrize("N", [17, 33, 35, 62, 130, 257, 513, 516])
def test_layer_rows_and_packed_rows_give_the_same_projection(qb, N):
    """The row quantizers' own GEMM format against packed rows, which the GEMM converts: the same bits, at rows that end
    inside a four, a block of 16 and a tile, with start values (512 and more) and without, and a ragged last group.  Rows of a NaN
    (all codes -8, the only way to that code), of an infinity, of zeros and of one value (codes 7) among them."""
    from paper_2604_17320_amd.model import KVCache4, make_taps
    d, H, Hkv, dh, F = 512 + 128, 10, 2, 64, 160
    W, L, cos, sin = build_gqa_layer(d, H, Hkv, dh, F, 77, 640)
    dkv = Hkv * dh
    x = wl.rng(N, "rows").standard_normal((N, d)).astype(np.float16)
    x[0, 5], x[N // 2, 9], x[N - 1], x[N - 2] = np.nan, np.inf, 0.0, 3.0
    xd, pos = dev(x), dev(np.arange(N, dtype=np.int32))
    t16 = lambda *s: torch.full(s, float("nan"), dtype=torch.float16, device="cuda")
    qkv, y, x_out = t16(N, d + 2 * dkv), t16(N, d + 2 * dkv), t16(N, d)
    cache, pos_out = KVCache4(1, N, Hkv, dh), torch.zeros(N, dtype=torch.int32, device="cuda")
    ws = torch.full((L.workspace_bytes(1, N),), 0xFF, dtype=torch.uint8, device="cuda")
    st = qb.State(1, N, 0, 0, xd.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    qb.quota_prefill_layer(L.desc, st, qb.KEEP_ALL, qb.quota_score_params_default(), cache.desc, make_taps(qkv=qkv), ws)
    codes, scale = torch.zeros((N, d // 2), dtype=torch.uint8, device="cuda"), torch.zeros(N, device="cuda")
    qb.quota_rmsnorm_quantize_act(xd, N, d, d, L.gamma1, W.eps, codes, scale)
    c = unpack4(host(codes))
    assert (c[0] == -8).all() and (c[N - 1] == 0).all() and c.max() == 7
    qb.quota_w4a4_gemm(codes, scale, N, L.qkv.desc, y, d + 2 * dkv)
    assert torch.equal(qkv.view(torch.int16), y.view(torch.int16))
    assert np.array_equal(host(y).view(np.uint16), oracle.w4a4_gemm(c, host(scale), *W.qkv).view(np.uint16))


@pytest.mark.parametrize("N", [130, 513])
@pytest.mark.parametrize("shape", [(512, 8, 4, 64, 1376), (256, 4, 4, 64, 32)])
def test_layer_on_tall_tiles_equals_the_same_on_short_ones(qb, pinned_gemm, shape, N):
    """The 128 x 256 tile's stages of two groups, one register set of weights between them, at an odd number of groups (11), at two
    and at one, against the 64 x 128 tile: the same bits, with start values (513 rows) and without."""
    from paper_2604_17320_amd.model import KVCache4, make_taps
    d, H, Hkv, dh, F = shape
    W, L, cos, sin = build_gqa_layer(d, H, Hkv, dh, F, 78, 640)
    x, pos = dev(wl.rng(N, "rows").standard_normal((N, d)).astype(np.float16)), dev(np.arange(N, dtype=np.int32))
    seen = []
    for variant in (4, 1):
        pinned_gemm(variant)
        qkv = torch.full((N, d + 2 * Hkv * dh), float("nan"), dtype=torch.float16, device="cuda")
        x_out = torch.full((N, d), float("nan"), dtype=torch.float16, device="cuda")
        cache, pos_out = KVCache4(1, N, Hkv, dh), torch.zeros(N, dtype=torch.int32, device="cuda")
        ws = torch.full((L.workspace_bytes(1, N),), 0xFF, dtype=torch.uint8, device="cuda")
        st = qb.State(1, N, 0, 0, x.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
        qb.quota_prefill_layer(L.desc, st, qb.KEEP_ALL, qb.quota_score_params_default(), cache.desc, make_taps(qkv=qkv), ws)
        seen.append((qkv, x_out))
    assert all(torch.equal(a.view(torch.int16), b.view(torch.int16)) and bool(a.isfinite().all()) for a, b in zip(*seen))


@pytest.mark.parametrize("N", [35, 515])
def test_layer_codes_at_half_steps(qb, N):
    """The layer's own quantizers round by a conversion to e4m3 where the public one adds 1.5 * 2^23: the same codes where a value
    lies half a step between two (ties go to the even code), next to it, and at zero from below; rows of a scale of every size
    among them.  O and down products of injected rows against the public quantizer and GEMM, with start values (515 rows) and without."""
    from paper_2604_17320_amd.model import KVCache4, make_taps
    d, H, Hkv, dh, F = 640, 10, 2, 64, 2080                    # five groups; sixteen and a ragged one, two chunks a thread
    W, L, cos, sin = build_gqa_layer(d, H, Hkv, dh, F, 79, 640)
    r = wl.rng(N, "half steps")

    def rows(n):
        a = np.exp2(r.integers(-9, 9, (N, 1))).astype(np.float64)
        x = r.integers(-14, 15, (N, n)) * a / 2                  # multiples of half a step, of maximum 7 a
        x[np.arange(N), r.integers(0, n, N)] = 7 * a[:, 0]
        near = r.random((N, n)) < 0.25
        x = np.where(near & (np.abs(x) < 7 * a), x * (1 + r.choice([-1, 1], (N, n)) * 2.0 ** -10), x)
        x[::5] = x[::5] * r.uniform(0.5, 1, (len(x[::5]), 1))
        x[1::7, ::3] = -1e-4 * a[1::7]
        return x.astype(np.float16)

    o, z, x = rows(d), rows(F), r.standard_normal((N, d)).astype(np.float16)
    xd, od, zd, pos = dev(x), dev(o), dev(z), dev(np.arange(N, dtype=np.int32))
    t16 = lambda *s: torch.full(s, float("nan"), dtype=torch.float16, device="cuda")
    x1, x_out = t16(N, d), t16(N, d)
    cache, pos_out = KVCache4(1, N, Hkv, dh), torch.zeros(N, dtype=torch.int32, device="cuda")
    ws = torch.full((L.workspace_bytes(1, N),), 0xFF, dtype=torch.uint8, device="cuda")
    st = qb.State(1, N, 0, 0, xd.data_ptr(), pos.data_ptr(), x_out.data_ptr(), pos_out.data_ptr())
    taps = make_taps(x1=x1, inject_o=od, inject_z=zd)
    qb.quota_prefill_layer(L.desc, st, qb.KEEP_ALL, qb.quota_score_params_default(), cache.desc, taps, ws)
    for rows_in, lin, res, got in ((o, L.o, xd, x1), (z, L.down, x1, x_out)):
        K = rows_in.shape[1]
        codes, scale, y = torch.zeros((N, K // 2), dtype=torch.uint8, device="cuda"), torch.zeros(N, device="cuda"), t16(N, d)
        qb.quota_quantize_act(dev(rows_in), N, K, K, codes, scale)
        want = oracle.quantize_act(rows_in)
        assert np.array_equal(unpack4(host(codes)), want[0])
        qb.quota_w4a4_gemm(codes, scale, N, lin.desc, y, d, res, d)
        assert torch.equal(got.view(torch.int16), y.view(torch.int16))
