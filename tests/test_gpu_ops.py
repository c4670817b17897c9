"""GPU parity, per operation, through the C ABI: the HIP path against the CPU
oracle on identical seeded inputs.  Integer outputs (int4 codes, int32
accumulators, index sets, KV codes, fp16 scales) must be bit-exact; fp16
tensors must be within 1e-2 relative (|a-b| <= 1e-2 * max(|b|, rms(b))) and
fp32 scores within 1e-5 relative."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_17320_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qb():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2604_17320_amd import binding
    binding.lib()
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def unpack4(p):
    """uint8 [..., n/2] nibble-packed (element 2j in the low nibble) -> int8 [..., n]."""
    p = np.asarray(p, np.uint8)
    out = np.empty(p.shape[:-1] + (p.shape[-1] * 2,), np.int16)
    out[..., 0::2] = p & 0xF
    out[..., 1::2] = p >> 4
    return ((out ^ 8) - 8).astype(np.int8)


def close_f16(a, b, tol=1e-2):
    a = a.astype(np.float64)
    b = b.astype(np.float64)
    rms = np.sqrt((b ** 2).mean()) if b.size else 0.0
    return np.all(np.abs(a - b) <= tol * np.maximum(np.abs(b), rms))


# ---------------------------------------------------------------- weights
@pytest.mark.parametrize("N,K", [(64, 1376), (128, 512), (192, 4096)])
def test_quantize_and_pack_weights(qb, N, K):
    from paper_2604_17320_amd.model import PackedLinear
    w = (wl.rng(3, "w", N, K).standard_normal((N, K), dtype=np.float32) * np.float32(0.02))
    w[1, :128] = 0
    codes, scales = oracle.quantize_weights(w)
    lin = PackedLinear.from_fp32(dev(w), keep_plain=True)
    assert np.array_equal(host(lin.codes), codes)
    assert np.array_equal(host(lin.plain_scales).view(np.uint16), scales.view(np.uint16))
    # packed layout: [group][row][64 bytes], zero padded; scales [group][row]
    G = (K + 127) // 128
    pk = unpack4(host(lin.packed).reshape(G, N, 64))
    full = np.zeros((N, G * 128), np.int8)
    full[:, :K] = codes
    assert np.array_equal(pk, full.reshape(N, G, 128).transpose(1, 0, 2))
    assert np.array_equal(host(lin.scales).reshape(G, N).view(np.uint16), scales.T.view(np.uint16))


@pytest.mark.parametrize("N,K", [(64, 32), (64, 1376), (192, 4096), (576, 11008), (128, 160)])
def test_one_pass_weight_packing_equals_the_two_calls(qb, N, K):
    from paper_2604_17320_amd.model import PackedLinear
    w = wl.rng(4, "w", N, K).standard_normal((N, K), dtype=np.float32) * np.float32(0.02)
    w[1, :128] = 0
    w[N - 1, K - 1] = 1e-9
    w[2, :32] = 3.5 * np.arange(-16, 16)                # ties of the rounding
    one, two = PackedLinear.from_fp32(dev(w)), PackedLinear.from_fp32(dev(w), keep_plain=True)
    assert torch.equal(one.packed, two.packed) and torch.equal(one.scales, two.scales)
    off = dev(np.concatenate([np.zeros(1, np.float32), w.ravel()]))[1:].view(N, K)      # not 16-byte aligned
    three = PackedLinear.from_fp32(off)
    assert torch.equal(three.packed, two.packed) and torch.equal(three.scales, two.scales)


def test_pack_weights_rejects_bad_shapes(qb):
    W = qb.Weights(48, 512, 1, 1)
    z = torch.zeros(8, dtype=torch.int8, device="cuda")
    s = torch.zeros(8, dtype=torch.float16, device="cuda")
    with pytest.raises(qb.QuotaError) as e:
        qb.quota_pack_weights(z, s, W)
    assert e.value.code == qb.ERR_SHAPE
    W = qb.Weights(64, 500, 1, 1)
    with pytest.raises(qb.QuotaError):
        qb.quota_pack_weights(z, s, W)


# ------------------------------------------------------------ quantizers
def _act(M, d, seed, scale=1.0):
    x = wl.rng(seed, "act", M, d).standard_normal((M, d), dtype=np.float32) * np.float32(scale)
    x[:, :: max(1, d // 7)] *= 20
    return x.astype(np.float16)


@pytest.mark.parametrize("M,d", [(80, 512), (37, 1376), (640, 4096), (5, 11008), (3, 16384), (1, 8), (5, 18944), (2, 32768)])
def test_quantize_act_bit_exact(qb, M, d):
    x = _act(M, d, 11)
    if M > 2:
        x[2] = 0
    q, s, ss, rs = oracle.quantize_act(x)
    xd = dev(x)
    qp = torch.empty((M, d // 2), dtype=torch.uint8, device="cuda")
    sc = torch.empty(M, dtype=torch.float32, device="cuda")
    sq = torch.empty(M, dtype=torch.float32, device="cuda")
    rq = torch.empty(M, dtype=torch.float32, device="cuda")
    qb.quota_quantize_act(xd, M, d, d, qp, sc, sq, rq)
    assert np.array_equal(unpack4(host(qp)), q)
    assert np.array_equal(host(sc), s)
    assert np.array_equal(host(sq), ss) and np.array_equal(host(rq), rs)
    # without the side outputs (other kernel instantiation), and with a row stride
    qp2 = torch.zeros_like(qp)
    sc2 = torch.zeros_like(sc)
    if d % 16 == 0:
        qb.quota_quantize_act(xd, M, d // 2, d, qp2, sc2)
        q2, s2, _, _ = oracle.quantize_act(x[:, : d // 2])
        assert np.array_equal(unpack4(host(qp2).reshape(-1)[: M * d // 4].reshape(M, d // 4)), q2)
        assert np.array_equal(host(sc2), s2)


def test_quantize_act_errors(qb):
    x = torch.zeros((4, 64), dtype=torch.float16, device="cuda")
    q = torch.zeros((4, 32), dtype=torch.uint8, device="cuda")
    s = torch.zeros(4, dtype=torch.float32, device="cuda")
    for args, code in [((x, 4, 60, 64, q, s), qb.ERR_SHAPE), ((x, 4, 64, 32, q, s), qb.ERR_SHAPE),
                       ((x, -1, 64, 64, q, s), qb.ERR_INVALID_ARG), ((None, 4, 64, 64, q, s), qb.ERR_NULL),
                       ((x, 4, 32776, 32776, q, s), qb.ERR_SHAPE)]:
        with pytest.raises(qb.QuotaError) as e:
            qb.quota_quantize_act(*args)
        assert e.value.code == code
    qb.quota_quantize_act(x, 0, 64, 64, q, s)          # empty input is fine


@pytest.mark.parametrize("M,d", [(80, 512), (33, 4096), (6, 5120), (3, 18944)])
def test_rmsnorm_quantize_act(qb, M, d):
    x = _act(M, d, 12, 1.7)
    gamma = wl.rng(12, "gamma", d).uniform(0.5, 1.5, d).astype(np.float32)
    h = oracle.rmsnorm(x, gamma, 1e-5)
    q, s, _, _ = oracle.quantize_act(h)
    _, _, ss, rs = oracle.quantize_act(x)
    qp = torch.empty((M, d // 2), dtype=torch.uint8, device="cuda")
    sc, sq, rq = (torch.empty(M, dtype=torch.float32, device="cuda") for _ in range(3))
    hh = torch.empty((M, d), dtype=torch.float16, device="cuda")
    qb.quota_rmsnorm_quantize_act(dev(x), M, d, d, dev(gamma), 1e-5, qp, sc, sq, rq, hh)
    assert np.array_equal(host(hh).view(np.uint16), h.view(np.uint16))
    assert np.array_equal(unpack4(host(qp)), q) and np.array_equal(host(sc), s)
    assert np.array_equal(host(sq), ss) and np.array_equal(host(rq), rs)
    qp2 = torch.empty_like(qp)
    sc2 = torch.empty_like(sc)
    qb.quota_rmsnorm_quantize_act(dev(x), M, d, d, dev(gamma), 1e-5, qp2, sc2)
    assert torch.equal(qp2, qp) and torch.equal(sc2, sc)


@pytest.mark.parametrize("d,eps", [(512, 0.0), (4096, 1e-5), (6144, 1e-30)])
def test_rmsnorm_of_rows_without_a_finite_scale(qb, d, eps):
    """Rows of zeros, of the smallest and the largest numbers, with an infinity and with a NaN: 1 / sqrt(mean + eps) as the definition gives
    it, infinite, zero and NaN included."""
    x = np.zeros((6, d), np.float16)
    x[1] = 6e-8
    x[2] = 65504
    x[3] = _act(1, d, 31, 1.0)
    x[4:] = x[3]
    x[4, 5], x[5, d - 1] = np.inf, np.nan
    gamma = wl.rng(31, "gamma", d).uniform(0.5, 1.5, d).astype(np.float32)
    f = x.astype(np.float32)
    with np.errstate(all="ignore"):
        rn = (1.0 / np.sqrt((f.astype(np.float64) ** 2).mean(1) + np.float64(np.float32(eps)))).astype(np.float32)
        h = (f * rn[:, None] * gamma).astype(np.float16)
        a = np.fmax.reduce(np.abs(h.astype(np.float32)), axis=1, initial=0.0)
        s = np.where(a == 0, np.float32(1), a / np.float32(7))
        t = h.astype(np.float32) * np.where(a == 0, np.float32(0), np.float32(7) / a)[:, None]
        q = np.where(np.isnan(t), -8, np.clip(np.rint(t), -8, 7)).astype(np.int8)
    qp = torch.empty((6, d // 2), dtype=torch.uint8, device="cuda")
    sc = torch.empty(6, dtype=torch.float32, device="cuda")
    hh = torch.empty((6, d), dtype=torch.float16, device="cuda")
    qb.quota_rmsnorm_quantize_act(dev(x), 6, d, d, dev(gamma), eps, qp, sc, None, None, hh)
    assert np.array_equal(host(hh), h, equal_nan=True)
    assert np.array_equal(host(sc), s) and np.array_equal(unpack4(host(qp)), q)


def test_quantize_act_of_every_absmax(qb):
    """Rows whose largest magnitude is each fp16 number once, infinity included: scales and codes are those of the two divisions, bit by bit."""
    M, d = 0x7c01, 64
    a = np.arange(M, dtype=np.uint16).view(np.float16).astype(np.float32)
    x = (a[:, None] * wl.rng(37, "every absmax").uniform(-1, 1, (M, d)).astype(np.float32)).astype(np.float16)
    x[:, 7] = a
    x[M - 1, 8:] = 1
    with np.errstate(all="ignore"):
        s = np.where(a == 0, np.float32(1), a / np.float32(7))
        inv = np.where(a == 0, np.float32(0), np.float32(7) / a)
        t = x.astype(np.float32) * inv[:, None]
        q = np.where(np.isnan(t), -8, np.clip(np.rint(t), -8, 7)).astype(np.int8)
    qp = torch.empty((M, d // 2), dtype=torch.uint8, device="cuda")
    sc = torch.empty(M, dtype=torch.float32, device="cuda")
    qb.quota_quantize_act(dev(x), M, d, d, qp, sc)
    assert np.array_equal(host(sc), s) and np.array_equal(unpack4(host(qp)), q)


@pytest.mark.parametrize("M,F", [(35, 1376), (9, 11008), (7, 18944), (2, 32768)])
def test_silu_mul_quantize_act(qb, M, F):
    gu = (_act(M, 2 * F, 13, 1.5))
    z = oracle.silu_mul(gu, F)
    q, s, _, _ = oracle.quantize_act(z)
    qp = torch.empty((M, F // 2), dtype=torch.uint8, device="cuda")
    sc = torch.empty(M, dtype=torch.float32, device="cuda")
    zz = torch.empty((M, F), dtype=torch.float16, device="cuda")
    qb.quota_silu_mul_quantize_act(dev(gu), M, F, qp, sc, zz)
    zg = host(zz)
    assert close_f16(zg, z)
    assert (zg.view(np.uint16) != z.view(np.uint16)).mean() < 5e-3      # fp32 vs fp64 silu
    # teacher-forced: with the oracle's z injected the codes are bit-exact
    qb.quota_silu_mul_quantize_act(dev(gu), M, F, qp, sc, None, dev(z))
    assert np.array_equal(unpack4(host(qp)), q) and np.array_equal(host(sc), s)


@pytest.mark.parametrize("M,d", [(2047, 6144), (2048, 6144), (2049, 6160), (2050, 4112), (2048, 1040), (4, 8192), (4, 8208)])
def test_row_kernels_at_the_edges_of_their_caches(qb, M, d):
    """Rows that just fill, and just miss, each register cache of a wave or workgroup, on both sides of the row count
    that tells them apart."""
    test_quantize_act_bit_exact(qb, M, d)
    test_rmsnorm_quantize_act(qb, M, d)
    test_silu_mul_quantize_act(qb, M, d)


# ------------------------------------------------------------------ GEMM
def _gemm_case(M, N, K, seed):
    r = wl.rng(seed, "gemm", M, N, K)
    w = r.standard_normal((N, K), dtype=np.float32) * np.float32(0.02)
    qw, sw = oracle.quantize_weights(w)
    x = _act(M, K, seed + 1)
    qa, sa, _, _ = oracle.quantize_act(x)
    res = r.standard_normal((M, N), dtype=np.float32).astype(np.float16)
    return qa, sa, qw, sw, res


def _pack4(codes):
    c = codes.astype(np.uint8) & 0xF
    return (c[..., 0::2] | (c[..., 1::2] << 4)).astype(np.uint8)


@pytest.mark.parametrize("M,N,K", [(80, 1536, 512), (35, 512, 1376), (300, 2752, 512), (129, 4096, 4096),
                                   (1, 64, 32), (640, 1536, 1376), (257, 320, 11008),
                                   (16, 4096, 4096), (7, 512, 1376), (16, 9216, 512), (13, 128, 11008)])
def test_w4a4_gemm_bit_exact(qb, M, N, K):
    from paper_2604_17320_amd.model import PackedLinear
    qa, sa, qw, sw, res = _gemm_case(M, N, K, 21)
    y_ref, acc_ref = oracle.w4a4_gemm(qa, sa, qw, sw, want_acc=True)
    yr_ref = oracle.w4a4_gemm(qa, sa, qw, sw, residual=res)
    lin = PackedLinear.from_codes(dev(qw), dev(sw))
    qad, sad = dev(_pack4(qa)), dev(sa)
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    acc = torch.empty((M, N), dtype=torch.int32, device="cuda")
    qb.quota_w4a4_gemm(qad, sad, M, lin.desc, y, N)                     # fast kernel
    assert np.array_equal(host(y).view(np.uint16), y_ref.view(np.uint16))
    y2 = torch.empty((M, N + 8), dtype=torch.float16, device="cuda")
    qb.quota_w4a4_gemm(qad, sad, M, lin.desc, y2, N + 8, dev(res), N, acc)   # residual + int32 debug
    assert np.array_equal(host(acc), acc_ref)
    assert np.array_equal(host(y2)[:, :N].view(np.uint16), yr_ref.view(np.uint16))
    y3 = torch.empty((M, N), dtype=torch.float16, device="cuda")
    qb.quota_w4a4_gemm(qad, sad, M, lin.desc, y3, N, dev(res), N)
    assert np.array_equal(host(y3).view(np.uint16), yr_ref.view(np.uint16))


@pytest.mark.parametrize("M,N,K", [(16, 4096, 1024), (9, 4160, 1024), (3, 8192, 992), (5, 8256, 1024), (12, 8192, 1056), (16, 64, 1024)])
def test_w4a4_gemm_of_few_short_rows(qb, M, N, K):
    """At most 16 rows of at most 1024 channels and 8192 columns, and just past each."""
    test_w4a4_gemm_bit_exact(qb, M, N, K)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
def test_w4a4_gemm_every_tile_bit_exact(qb, tile, pinned_gemm):
    """Each of the five tile instantiations, pinned with quota_set_gemm_variant, on shapes with ragged
    rows, a ragged last group and several column tiles."""
    from paper_2604_17320_amd.model import PackedLinear
    pinned_gemm(tile)
    for M, N, K in [(150, 1024, 1376), (70, 512, 4096)]:
        qa, sa, qw, sw, res = _gemm_case(M, N, K, 23)
        y_ref = oracle.w4a4_gemm(qa, sa, qw, sw, residual=res)
        lin = PackedLinear.from_codes(dev(qw), dev(sw))
        y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        qb.quota_w4a4_gemm(dev(_pack4(qa)), dev(sa), M, lin.desc, y, N, dev(res), N)
        assert np.array_equal(host(y).view(np.uint16), y_ref.view(np.uint16)), (tile, M, N, K)


@pytest.mark.parametrize("M,N,K", [(257, 21952, 416), (641, 10944, 160), (513, 12224, 1056)])
def test_w4a4_gemm_on_the_tile_of_packed_rows(qb, M, N, K):
    """The 64 x 256 tile, which only the choice takes: ragged rows, columns that end inside a tile, two to nine groups, the last one
    ragged, in stages of two; with a residual and without."""
    from paper_2604_17320_amd.model import PackedLinear
    qa, sa, qw, sw, res = _gemm_case(M, N, K, 24)
    lin, qad, sad = PackedLinear.from_codes(dev(qw), dev(sw)), dev(_pack4(qa)), dev(sa)
    y, yr = (torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    qb.quota_profile_begin(8)
    qb.quota_w4a4_gemm(qad, sad, M, lin.desc, y, N)
    qb.quota_w4a4_gemm(qad, sad, M, lin.desc, yr, N, dev(res), N)
    assert qb.quota_profile_collect()["w4a4_gemm_64x256"]["launches"] == 2
    assert np.array_equal(host(y).view(np.uint16), oracle.w4a4_gemm(qa, sa, qw, sw).view(np.uint16))
    assert np.array_equal(host(yr).view(np.uint16), oracle.w4a4_gemm(qa, sa, qw, sw, residual=res).view(np.uint16))


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("off", [1, 4, 8])
def test_w4a4_gemm_output_and_residual_at_any_element(qb, tile, off, pinned_gemm):
    """Rows of y and residual that start at any element, an odd number of elements apart; what lies between them stays."""
    from paper_2604_17320_amd.model import PackedLinear
    pinned_gemm(tile)
    M, N, K = 70, 320, 416
    qa, sa, qw, sw, res = _gemm_case(M, N, K, 25)
    lin = PackedLinear.from_codes(dev(qw), dev(sw))
    ldy, ldr = N + 3, N + 5
    y = torch.full((off + M * ldy,), 7.0, dtype=torch.float16, device="cuda")
    r = torch.zeros(off + M * ldr, dtype=torch.float16, device="cuda")
    rows = lambda t, ld: t[off:].view(M, ld)
    rows(r, ldr)[:, :N] = dev(res)
    qb.quota_w4a4_gemm(dev(_pack4(qa)), dev(sa), M, lin.desc, y[off:], ldy, r[off:], ldr)
    ref = oracle.w4a4_gemm(qa, sa, qw, sw, residual=res)
    assert np.array_equal(host(rows(y, ldy)[:, :N].contiguous()).view(np.uint16), ref.view(np.uint16))
    assert bool((rows(y, ldy)[:, N:] == 7.0).all()) and bool((y[:off] == 7.0).all())


@pytest.mark.parametrize("M", [1, 16, 17, 45, 160])
def test_w4a4_gemm_with_scales_at_an_odd_halfword(qb, M):
    """Weight scales that start between two dwords: the bits of the aligned call, output and integer sums."""
    from paper_2604_17320_amd.model import PackedLinear
    N, K = 192, 416
    q, s, qw, sw, res = _gemm_case(M, N, K, 31)
    lin = PackedLinear.from_codes(dev(qw), dev(sw))
    room = torch.cat([lin.scales.new_zeros(1), lin.scales])
    odd = qb.Weights(N, K, lin.packed.data_ptr(), room[1:].data_ptr())
    assert odd.scales % 4 == 2
    outs = []
    for W in (lin.desc, odd):
        y, yr, ya = (torch.zeros((M, N), dtype=torch.float16, device="cuda") for _ in range(3))
        acc, alone = (torch.zeros((M, N), dtype=torch.int32, device="cuda") for _ in range(2))
        qad, sad, resd = dev(_pack4(q)), dev(s), dev(res)
        args = (qad, sad, M, W)
        qb.quota_w4a4_gemm(*args, y, N)
        qb.quota_w4a4_gemm(*args, yr, N, resd, N)
        qb.quota_w4a4_gemm(*args, ya, N, acc_i32=acc)
        qb.quota_w4a4_gemm(*args, None, N, acc_i32=alone)
        outs.append([t.view(torch.int16) for t in (y, yr, ya)] + [acc, alone])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    assert torch.equal(outs[0][0], outs[0][2])


def test_w4a4_gemm_unit_scales_give_exact_integers(qb):
    from paper_2604_17320_amd.model import PackedLinear
    r = wl.rng(5, "unit")
    M, N, K = 70, 128, 256
    qa = r.integers(-8, 8, (M, K)).astype(np.int8)
    qw = r.integers(-8, 8, (N, K)).astype(np.int8)
    lin = PackedLinear.from_codes(dev(qw), dev(np.ones((N, 2), np.float16)))
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    qb.quota_w4a4_gemm(dev(_pack4(qa)), dev(np.ones(M, np.float32)), M, lin.desc, y, N)
    exact = qa.astype(np.int64) @ qw.astype(np.int64).T       # |sum| <= 16384: one fp16 rounding
    assert np.array_equal(host(y), exact.astype(np.float16))


# -------------------------------------------------------- RoPE + KV quant
@pytest.mark.parametrize("H,dh,M", [(8, 64, 80), (32, 128, 70), (3, 128, 5)])
def test_rope_kv_quant_bit_exact(qb, H, dh, M):
    d = H * dh
    qkv = _act(M, 3 * d, 31, 2.0)
    qkv[3, d:d + 64] = 0
    n_pos = 700
    pos = wl.rng(31, "pos").integers(0, n_pos, M).astype(np.int32)
    cos, sin = wl.rope_tables(dh, n_pos)
    q_ref = oracle.rope(qkv[:, :d], H, dh, pos, cos, sin)
    k_ref = oracle.rope(qkv[:, d:2 * d], H, dh, pos, cos, sin)
    kc, ks, khat = oracle.kv_quant(k_ref)
    vc, vs, vhat = oracle.kv_quant(np.ascontiguousarray(qkv[:, 2 * d:]))
    f16 = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda")
    u8 = lambda *s: torch.empty(s, dtype=torch.uint8, device="cuda")
    q_rot, kh, vh = f16(M, d), f16(M, d), f16(M, d)
    kcd, vcd, ksd, vsd = u8(M, d // 2), u8(M, d // 2), f16(M, d // 64), f16(M, d // 64)
    qb.quota_rope_kv_quant(dev(qkv), M, H, dh, dev(pos), dev(cos), dev(sin), n_pos, q_rot, kh, vh,
                           kcd, ksd, vcd, vsd)
    assert np.array_equal(host(q_rot).view(np.uint16), q_ref.view(np.uint16))
    assert np.array_equal(unpack4(host(kcd)), kc) and np.array_equal(unpack4(host(vcd)), vc)
    assert np.array_equal(host(ksd).view(np.uint16), ks.view(np.uint16))
    assert np.array_equal(host(vsd).view(np.uint16), vs.view(np.uint16))
    assert np.array_equal(host(kh).view(np.uint16), khat.view(np.uint16))
    assert np.array_equal(host(vh).view(np.uint16), vhat.view(np.uint16))


def test_kv_quant_of_every_group_maximum(qb):
    """The quantizer's scale and reciprocal are made without IEEE divisions: bit-exact for each of the 31744 finite fp16
    maxima a group can have, zero and the subnormals included."""
    H, dh = 64, 128
    d = H * dh
    top = np.arange(31744, dtype=np.uint16).view(np.float16).reshape(-1, d // 64, 1).astype(np.float32)
    M = top.shape[0]
    r = wl.rng(40, "groups")
    part = r.uniform(-1, 1, (M, d // 64, 64))
    part[:, :, ::4] = np.round(part[:, :, ::4] * 14) / 14            # multiples of half a step
    part[np.arange(M)[:, None], np.arange(d // 64)[None], r.integers(0, 64, (M, d // 64))] = 1.0
    v = (top * part).astype(np.float16).reshape(M, d)
    codes, scales, vhat = oracle.kv_quant(v)
    qkv = np.concatenate([np.zeros_like(v), np.zeros_like(v), v], axis=1)
    f16 = lambda *shape: torch.empty(shape, dtype=torch.float16, device="cuda")
    q8 = lambda: torch.empty((M, d // 2), dtype=torch.uint8, device="cuda")
    out = dict(q=f16(M, d), k=f16(M, d), v=f16(M, d), kc=q8(), ks=f16(M, d // 64), vc=q8(), vs=f16(M, d // 64))
    cos, sin = wl.rope_tables(dh, 1)
    qb.quota_rope_kv_quant(dev(qkv), M, H, dh, torch.zeros(M, dtype=torch.int32, device="cuda"), dev(cos), dev(sin), 1,
                           out["q"], out["k"], out["v"], out["kc"], out["ks"], out["vc"], out["vs"])
    assert np.array_equal(host(out["vs"]).view(np.uint16), scales.view(np.uint16))
    assert np.array_equal(unpack4(host(out["vc"])), codes)
    assert np.array_equal(host(out["v"]).view(np.uint16), vhat.view(np.uint16))


def test_kv_quant_of_groups_that_are_not_finite(qb):
    """Groups whose maximum is infinite (finite values become 0, infinities NaN and so -8), with a NaN beside finite values (the maximum
    passes over it, its code is -8) and of NaNs alone: codes, scales and dequantized values as the definition gives them."""
    from paper_2604_17320_amd.model import KVCache4
    M, H, dh = 9, 2, 128
    d = H * dh
    r = wl.rng(41, "not finite")
    v = r.standard_normal((M, d)).astype(np.float16)
    bad = np.array([np.inf, -np.inf, np.nan], np.float16)
    for row in range(1, M):                              # row 0 stays finite
        for g in range(d // 64):
            v[row, 64 * g + r.permutation(64)[: row]] = bad[r.integers(0, 3, row)] if row > 3 else bad[row - 1]
    v[M - 1, :64] = np.nan
    x = v.astype(np.float32).reshape(M, d // 64, 64)
    a = np.fmax.reduce(np.abs(x), axis=2, initial=0.0)
    scales = (a / np.float32(7)).astype(np.float16)
    scales[scales == 0] = 1
    s = scales.astype(np.float32)[:, :, None]
    with np.errstate(invalid="ignore"):
        t = x * (np.float32(1) / s)
        codes = np.where(np.isnan(t), -8, np.clip(np.rint(t), -8, 7)).astype(np.float32)
        hat = (codes * s).astype(np.float16).reshape(M, d)
    codes = codes.astype(np.int8).reshape(M, d)
    assert np.array_equal(codes[0], oracle.kv_quant(v[:1])[0][0]) and (codes[M - 1, :64] == -8).all()
    qkv = np.concatenate([np.zeros_like(v), np.zeros_like(v), v], axis=1)
    f16 = lambda *shape: torch.zeros(shape, dtype=torch.float16, device="cuda")
    q8 = lambda: torch.zeros((M, d // 2), dtype=torch.uint8, device="cuda")
    out = dict(q=f16(M, d), k=f16(M, d), v=f16(M, d), kc=q8(), ks=f16(M, d // 64), vc=q8(), vs=f16(M, d // 64))
    cos, sin = wl.rope_tables(dh, 1)
    qb.quota_rope_kv_quant(dev(qkv), M, H, dh, torch.zeros(M, dtype=torch.int32, device="cuda"), dev(cos), dev(sin), 1,
                           out["q"], out["k"], out["v"], out["kc"], out["ks"], out["vc"], out["vs"])
    cache = KVCache4(1, M, H, dh)
    qb.quota_kv_quant_append(dev(v), dev(v), 1, M, H, dh, None, M, cache.desc)
    for got_codes, got_scales in ((out["vc"], out["vs"]), (cache.k_codes[0], cache.k_scales[0]), (cache.v_codes[0], cache.v_scales[0])):
        assert np.array_equal(unpack4(host(got_codes)), codes)
        assert np.array_equal(host(got_scales).view(np.uint16), scales.view(np.uint16))
    assert np.array_equal(host(out["v"]), hat, equal_nan=True)


def test_kv_quant_append(qb):
    from paper_2604_17320_amd.model import KVCache4
    B, N, H, dh = 2, 24, 4, 128
    d = H * dh
    k = _act(B * N, d, 41, 2.0)
    v = _act(B * N, d, 42, 0.7)
    kc, ks, _ = oracle.kv_quant(k)
    vc, vs, _ = oracle.kv_quant(v)
    cache = KVCache4(B, 20, H, dh)
    rows = np.stack([np.sort(wl.rng(41, "rows", b).permutation(N)[:7]) for b in range(B)]).astype(np.int32)
    qb.quota_kv_quant_append(dev(k), dev(v), B, N, H, dh, None, 5, cache.desc)      # rows 0..4
    qb.quota_kv_quant_append(dev(k), dev(v), B, N, H, dh, dev(rows), 7, cache.desc)
    assert cache.len == 12
    for b in range(B):
        src = np.concatenate([np.arange(5), rows[b]]) + b * N
        assert np.array_equal(unpack4(host(cache.k_codes)[b, :12]), kc[src])
        assert np.array_equal(unpack4(host(cache.v_codes)[b, :12]), vc[src])
        assert np.array_equal(host(cache.k_scales)[b, :12].view(np.uint16), ks[src].view(np.uint16))
        assert np.array_equal(host(cache.v_scales)[b, :12].view(np.uint16), vs[src].view(np.uint16))
    with pytest.raises(qb.QuotaError) as e:
        qb.quota_kv_quant_append(dev(k), dev(v), B, N, H, dh, None, 9, cache.desc)
    assert e.value.code == qb.ERR_CAPACITY and cache.len == 12
    qb.quota_kv_quant_append(dev(k), dev(v), B, N, H, dh, None, 0, cache.desc)
    assert cache.len == 12


# ------------------------------------------------------------- attention
@pytest.mark.parametrize("B,N,H,dh,vb,Nv", [(1, 80, 8, 64, 0, 64), (2, 200, 3, 128, 5, 150),
                                             (1, 640, 4, 128, 0, 576), (1, 33, 2, 128, 0, 0)])
def test_attention_prefill_and_column_masses(qb, B, N, H, dh, vb, Nv):
    d = H * dh
    q = _act(B * N, d, 51, 1.0)
    _, _, khat = oracle.kv_quant(_act(B * N, d, 52, 1.0))
    _, _, vhat = oracle.kv_quant(_act(B * N, d, 53, 1.0))
    o_ref, ci_ref, cv_ref = oracle.attention(q, khat, vhat, B, N, H, dh, vb, Nv)
    o = torch.empty((B * N, d), dtype=torch.float16, device="cuda")
    ci = torch.zeros((B, max(Nv, 1)), dtype=torch.float32, device="cuda")
    cv = torch.zeros((B, max(Nv, 1)), dtype=torch.float32, device="cuda")
    ws = torch.empty(qb.quota_attention_workspace_bytes(B, N, H, dh), dtype=torch.uint8, device="cuda")
    qb.quota_attention_prefill(dev(q), dev(khat), dev(vhat), B, N, H, dh, vb, Nv, o, ci, cv, ws)
    assert close_f16(host(o), o_ref)
    if Nv:
        cig, cvg = host(ci)[:, :Nv], host(cv)[:, :Nv]
        assert np.allclose(cig, ci_ref, rtol=2e-5, atol=1e-7), np.abs(cig / ci_ref - 1).max()
        assert np.allclose(cvg, cv_ref, rtol=2e-5, atol=1e-7), np.abs(cvg / cv_ref - 1).max()


# two groups of waves take the query tiles in turn: one tile only, an odd number, keys that begin inside a tile, and past 256
# workgroups of few tiles a single group
@pytest.mark.parametrize("B,N,H,dh,vb,Nv", [(1, 64, 2, 128, 0, 64), (1, 33, 1, 64, 5, 20), (1, 193, 2, 64, 3, 150),
                                             (1, 333, 2, 128, 200, 133), (1, 65, 3, 128, 64, 1), (3, 200, 90, 64, 0, 200)])
def test_column_masses_by_groups(qb, B, N, H, dh, vb, Nv):
    d = H * dh
    q = _act(B * N, d, 54, 1.0)
    _, _, khat = oracle.kv_quant(_act(B * N, d, 55, 1.0))
    _, _, vhat = oracle.kv_quant(_act(B * N, d, 56, 1.0))
    o_ref, ci_ref, cv_ref = oracle.attention(q, khat, vhat, B, N, H, dh, vb, Nv)
    o = torch.empty((B * N, d), dtype=torch.float16, device="cuda")
    ci, cv = (torch.full((B, Nv), -1.0, dtype=torch.float32, device="cuda") for _ in range(2))
    ws = torch.empty(qb.quota_attention_workspace_bytes(B, N, H, dh), dtype=torch.uint8, device="cuda")
    qb.quota_attention_prefill(dev(q), dev(khat), dev(vhat), B, N, H, dh, vb, Nv, o, ci, cv, ws)
    assert close_f16(host(o), o_ref)
    assert np.allclose(host(ci), ci_ref, rtol=2e-5, atol=1e-7)
    assert np.allclose(host(cv), cv_ref, rtol=2e-5, atol=1e-7)


# (from 512 tokens on a launch of more than 512 workgroups, one per head and 128 visual keys, has one group of waves a workgroup, before from
# 256; the sequence alone has two groups)
@pytest.mark.parametrize("N,H,dh,vb,Nv,B", [(300, 8, 64, 14, 250, 17), (193, 6, 128, 0, 193, 22), (520, 8, 64, 60, 390, 17),
                                            (643, 8, 128, 3, 577, 13), (705, 6, 64, 100, 600, 18)])
def test_cues_of_a_sequence_do_not_depend_on_the_others(qb, N, H, dh, vb, Nv, B):
    """The masses of a sequence in a batch have the bits of the same sequence alone, whichever form of the cue pass a launch takes."""
    d, per = H * dh, H * ((Nv + 127) // 128)
    most = 512 if N >= 512 else 256
    assert per <= most < per * B                     # (the two forms)
    q = dev(_act(B * N, d, 64, 1.0))
    khat, vhat = (dev(oracle.kv_quant(_act(B * N, d, seed, 1.0))[2]) for seed in (65, 66))

    def cues(first, n):
        rows = slice(first * N, (first + n) * N)
        o = torch.empty((n * N, d), dtype=torch.float16, device="cuda")
        ci, cv = (torch.full((n, Nv), -1.0, dtype=torch.float32, device="cuda") for _ in range(2))
        ws = torch.empty(qb.quota_attention_workspace_bytes(n, N, H, dh), dtype=torch.uint8, device="cuda")
        qb.quota_attention_prefill(q[rows], khat[rows], vhat[rows], n, N, H, dh, vb, Nv, o, ci, cv, ws)
        return host(ci), host(cv)
    batch = cues(0, B)
    for b in (0, B // 2, B - 1):
        for got, alone in zip(batch, cues(b, 1)):
            assert np.array_equal(got[b].view(np.uint32), alone[0].view(np.uint32))


# (workgroups of two waves up to 160 of four, one per head and 128 queries or visual keys: the sequence alone; of four in the batch)
@pytest.mark.parametrize("N,H,Hkv,dh,vb,Nv,B", [(64, 8, 8, 64, 0, 64, 21), (65, 8, 2, 128, 1, 63, 21), (127, 8, 8, 64, 14, 65, 21), (129, 8, 8, 128, 0, 129, 11),
                                                (193, 6, 6, 128, 65, 128, 27), (640, 28, 4, 128, 30, 576, 2)])
def test_attention_of_two_and_of_four_waves(qb, N, H, Hkv, dh, vb, Nv, B):
    """Outputs and masses of a sequence have the same bits from workgroups of either width, and the outputs those of the reference."""
    d, dkv = H * dh, Hkv * dh
    for blocks in (H * ((N + 127) // 128), H * ((Nv + 127) // 128)):           # of the forward pass, of the cue pass
        assert blocks <= 160 < blocks * B
    q = _act(B * N, d, 74, 1.0)
    khat, vhat = (oracle.kv_quant(_act(B * N, dkv, seed, 1.0))[2] for seed in (75, 76))
    qd, kd, vd = dev(q), dev(khat), dev(vhat)

    def run(first, n):
        rows = slice(first * N, (first + n) * N)
        o = torch.full((n * N, d), float("nan"), dtype=torch.float16, device="cuda")
        ci, cv = (torch.full((n, Nv), -1.0, dtype=torch.float32, device="cuda") for _ in range(2))
        ws = torch.full((qb.quota_attention_workspace_bytes(n, N, H, dh),), 0xFF, dtype=torch.uint8, device="cuda")
        qb.quota_attention_prefill_gqa(qd[rows], kd[rows], vd[rows], n, N, H, Hkv, dh, vb, Nv, o, ci, cv, ws)
        return host(o).reshape(n, N * d), host(ci), host(cv)
    batch = run(0, B)
    for b in (0, B - 1):
        for got, alone in zip(batch, run(b, 1)):
            assert np.array_equal(got[b].view(np.uint8), alone[0].view(np.uint8))
    if H == Hkv:
        assert close_f16(batch[0][0].reshape(N, d), oracle.attention(q[:N], khat[:N], vhat[:N], 1, N, H, dh, vb, Nv)[0])


# -------------------------------------------------------- score and top-k
def _metrics(B, Nv, seed):
    r = wl.rng(seed, "metrics", B, Nv)
    return (r.uniform(100, 9000, (B, Nv)).astype(np.float32), r.uniform(1, 400, (B, Nv)).astype(np.float32),
            r.uniform(0, 0.2, (B, Nv)).astype(np.float32), r.uniform(0, 3, (B, Nv)).astype(np.float32))


@pytest.mark.parametrize("B,Nv", [(1, 64), (3, 576), (2, 2880), (1, 1), (1, 3072), (2, 7), (2, 4100), (1, 8192)])
def test_score_tokens_bit_exact(qb, B, Nv):
    ss, rs, ci, cv = _metrics(B, Nv, 61)
    if Nv > 4:
        cv[0] = 0.25                                    # a flat metric -> 0.5
        ci[0, :3] = ci[0, 3]                            # ties among the order statistics
    for kw in [dict(), dict(w_m=0.0, w_c=0.5333, w_s=0.1833, w_r=0.2833), dict(p_lo=0, p_hi=100),
               dict(p_lo=25, p_hi=50)]:
        sc_ref, g_ref = oracle.score(ss, rs, ci, cv, want_normed=True, **kw)
        p = qb.quota_score_params_default()
        for k, v in kw.items():
            setattr(p, {"p_lo": "pct_lo", "p_hi": "pct_hi"}.get(k, k), v)
        sc = torch.empty((B, Nv), dtype=torch.float32, device="cuda")
        g = torch.empty((4, B, Nv), dtype=torch.float32, device="cuda")
        qb.quota_score_tokens(dev(ss), dev(rs), dev(ci), dev(cv), B, Nv, p, sc, g)
        assert np.array_equal(host(g), g_ref)
        assert np.array_equal(host(sc), sc_ref)


@pytest.mark.parametrize("Nv", [1, 64, 65, 250, 1024, 1025])
def test_score_tokens_of_odd_metrics(qb, Nv):
    """Infinities, signed zeros, denormals and huge numbers among the metrics; squares whose roots are equal though they are not."""
    ss, rs, ci, cv = _metrics(2, Nv, 63)
    odd = np.array([0.0, -0.0, 1e-45, 3e38, np.inf, 1e-38], np.float32)
    for m in (ss, rs, ci, cv):
        m[0, : min(Nv, 6)] = odd[: min(Nv, 6)]
    ss[1] = np.float32(4.0) + np.arange(Nv, dtype=np.float32)[::-1] * np.float32(2.0 ** -21)
    sc_ref, g_ref = oracle.score(ss, rs, ci, cv, want_normed=True)
    sc = torch.empty((2, Nv), dtype=torch.float32, device="cuda")
    g = torch.empty((4, 2, Nv), dtype=torch.float32, device="cuda")
    qb.quota_score_tokens(dev(ss), dev(rs), dev(ci), dev(cv), 2, Nv, qb.quota_score_params_default(), sc, g)
    assert np.array_equal(host(g), g_ref, equal_nan=True) and np.array_equal(host(sc), sc_ref, equal_nan=True)


def test_score_tokens_from_hidden(qb):
    shape = wl.CONFIGS[0]
    x = wl.hidden_state(shape, 7)
    B, N, Nv, d = 1, shape.N, shape.Nv, shape.d
    _, _, ss, rs = oracle.quantize_act(x[:Nv])
    _, _, ci, cv = _metrics(B, Nv, 62)
    sc_ref = oracle.score(ss[None], rs[None], ci, cv)
    sc = torch.empty((B, Nv), dtype=torch.float32, device="cuda")
    ws = torch.empty(2 * B * Nv, dtype=torch.float32, device="cuda")
    qb.quota_score_tokens_from_hidden(dev(x), B, Nv, d, d, N * d, dev(ci), dev(cv),
                                      qb.quota_score_params_default(), sc, None, ws)
    assert np.array_equal(host(sc), sc_ref)


@pytest.mark.parametrize("B,Nv", [(1, 64), (3, 576), (2, 2880), (1, 3072), (2, 5), (2, 4100), (1, 8192)])
def test_topk_prune_bit_exact(qb, B, Nv):
    r = wl.rng(71, "topk", B, Nv)
    sc = (np.round(r.uniform(0, 1, (B, Nv)) * 50) / 50).astype(np.float32)     # plenty of ties
    if Nv > 10:
        sc[0, 5] = np.nan
        sc[0, 7] = -0.0
        sc[0, 8] = 0.0
    scd = dev(sc)
    for K in sorted({0, 1, 2, Nv // 3, int(np.ceil(0.3 * Nv)), Nv - 1, Nv, Nv + 9}):
        ref = oracle.topk(sc, K)
        k = min(K, Nv)
        out = torch.full((B, max(k, 1)), -1, dtype=torch.int32, device="cuda")
        qb.quota_topk_prune(scd, B, Nv, K, out)
        assert np.array_equal(host(out)[:, :k].reshape(B, k), ref), (Nv, K)
    allsame = dev(np.full((B, Nv), 0.5, np.float32))
    k = max(1, Nv // 2)
    out = torch.empty((B, k), dtype=torch.int32, device="cuda")
    qb.quota_topk_prune(allsame, B, Nv, k, out)
    assert np.array_equal(host(out), np.tile(np.arange(k, dtype=np.int32), (B, 1)))
    with pytest.raises(qb.QuotaError):
        qb.quota_topk_prune(scd, B, 8200, 3, out)


@pytest.mark.parametrize("close,copies", [(63, 1), (64, 1), (65, 1), (64, 4), (200, 1), (200, 150)])
def test_topk_prune_where_many_keys_share_their_digits(qb, close, copies):
    """Keys that agree in their first digits, around the 64 that one wave ranks and more, with ties among them."""
    r = wl.rng(72, "topk-close", close, copies)
    Nv = 500
    sc = np.concatenate([np.float32(0.75) + np.arange(close, dtype=np.float32) // copies * np.float32(2.0 ** -24),
                         r.uniform(-3e4, 3e4, Nv - close).astype(np.float32)])
    sc = r.permutation(sc).astype(np.float32)[None]
    above = int((sc > 0.8).sum())
    for K in (above, above + 1, above + close // 2, above + close - 1, above + close, above + close + 1):
        out = torch.full((1, K), -1, dtype=torch.int32, device="cuda")
        qb.quota_topk_prune(dev(sc), 1, Nv, K, out)
        assert np.array_equal(host(out), oracle.topk(sc, K))
