"""The weight-streaming GEMM of few rows, and the LN^quant fused in front of it: edges of its row blocks (16, 32) and column tiles
(16 columns, one to four tiles per workgroup, a last workgroup with fewer), one and several steps of K per wave, every operand type."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB, prep

SKINNY = 4                       # include/hero_debug.h
# M, N, K in bytes of the operands
SHAPES = [(1, 4096, 1024), (16, 4096, 1024), (17, 4112, 1024), (8, 8192, 1024), (32, 8208, 1024), (5, 12288, 1024), (31, 12272, 1024),
          (3, 1024, 4096), (9, 512, 8192), (24, 272, 16384), (2, 10256, 3072)]
DTYPES = [torch.int8, torch.float8_e4m3fn, torch.bfloat16, torch.float16]


@pytest.mark.parametrize("dt", DTYPES)
def test_route(dt):
    hero = pkg.load()
    k = lambda M, N, kb, **kw: hero.hero_gemm_kernel(dt, M, N, kb // dt.itemsize, **kw)
    for M, N, kb in SHAPES:
        assert k(M, N, kb) == SKINNY and k(M, N, kb, epi=HB.EPI_GELU_REQUANT) == SKINNY
        assert k(33, N, kb) != SKINNY                                # more rows
        assert k(M, N + 8, kb) != SKINNY                             # half a column tile
        assert k(M, N, kb + 128) != SKINNY                           # K the eight waves do not share evenly
    assert k(1, 2048, 1024) != SKINNY and k(1, 12304, 1024) != SKINNY
    if dt == torch.int8:
        assert k(1, 4096, 4096, epi=HB.EPI_RAW_I32) != SKINNY


@pytest.mark.parametrize("T,d,f,insists", [(1, 4096, 16384, False), (32, 4096, 16384, False), (33, 4096, 16384, True), (64, 4096, 16384, True),
                                            (16, 512, 16384, True), (16, 1024, 8192, False), (32, 1024, 16384, True), (1, 1024, 16384, False)])
def test_a_layer_insists_on_the_scratch_it_writes(T, d, f, insists):
    """A decode layer of few rows streams its weights without a K split: a workspace without the planes of one is accepted (the call
    goes on to the missing pointers), and refused where there are planes to write."""
    import types
    hero = pkg.load()
    desc = hero.layer_desc(HB.ARCH_PRE_LN, d, d // 128, 128, f, 1e-5, HB.MASK_CAUSAL, HB.MODE_M3)
    up = lambda n: (n + 255) // 256 * 256
    acts = sum(up(n) for n in (T * d, 4 * T, 3 * T * d, T * d, T * d, 4 * T, T * f))
    assert hero.hero_layer_workspace_bytes(desc, T, 1) > acts       # (what it can use keeps room for the split)
    raw = torch.empty(acts + 256, dtype=torch.uint8)
    ws = raw[-raw.data_ptr() % 256:][:acts]
    with pytest.raises(HB.HeroError) as e:
        hero.hero_layer_fwd(desc, HB.LayerWeights(), T, 1, ws, stream=types.SimpleNamespace(cuda_stream=0))
    assert e.value.status == (5 if insists else 1)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_int8(M, N, K):
    hero = pkg.load()
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a = torch.randint(-127, 128, (M, K + 16), device="cuda", generator=g, dtype=torch.int8)[:, :K]
    w = torch.randint(-127, 128, (N, K), device="cuda", generator=g, dtype=torch.int8)
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N + 1, device="cuda", generator=g)[1:] + 0.5) / (90 * K ** 0.5)
    bias = torch.randn(N, device="cuda", generator=g)
    res = torch.randn((M, N + 4), device="cuda", generator=g).to(torch.bfloat16)[:, :N]
    S = torch.rand(N, device="cuda", generator=g) / 30 + 0.02
    for row, b in ((rs, bias), (None, None)):
        # every other kernel gives the same bits (the integer sums are exact, the epilogue's order is one): the ring is forced
        kw = dict(a_row_scale=row, b_col_scale=cs, bias=b)
        for e in (dict(epi=HB.EPI_REQUANT, out_dtype=torch.int8), dict(epi=HB.EPI_DEQUANT, out_dtype=torch.float16),
                  dict(epi=HB.EPI_DEQUANT, out_dtype=torch.bfloat16, residual=res), dict(epi=HB.EPI_DEQUANT_GELU, out_dtype=torch.bfloat16),
                  dict(epi=HB.EPI_GELU_REQUANT, out_dtype=torch.int8, out_col_scale=S)):
            assert torch.equal(hero.hero_int8_gemm(a, w, **kw, **e), hero.hero_int8_gemm(a, w, **kw, **e, tile=2)), (row is None, e)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(8, 1024, 16384), (32, 1024, 16384), (17, 592, 12288), (24, 2048, 24576), (32, 1280, 16384), (16, 512, 9216)])
def test_with_scratch_for_a_split(M, N, K):
    """Few rows of a very long K, on either side of the rule that splits it where there is scratch: the same bits."""
    hero, g = pkg.load(), torch.Generator(device="cuda").manual_seed(K)
    a, w = (torch.randint(-127, 128, (n, K), device="cuda", generator=g, dtype=torch.int8) for n in (M, N))
    rs, cs, bias = torch.rand(M, device="cuda", generator=g) + 0.5, torch.rand(N, device="cuda", generator=g) / 9000, torch.randn(N, device="cuda", generator=g)
    ws = torch.full((hero.hero_int8_gemm_workspace_bytes(M, N, K),), 0xA5, dtype=torch.uint8, device="cuda")
    for e in (dict(epi=HB.EPI_DEQUANT, out_dtype=torch.bfloat16), dict(epi=HB.EPI_REQUANT, out_dtype=torch.int8)):
        assert torch.equal(hero.hero_int8_gemm(a, w, rs, cs, bias, workspace=ws, **e), hero.hero_int8_gemm(a, w, rs, cs, bias, **e))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,kb", SHAPES)
@pytest.mark.parametrize("dt", DTYPES[1:])
def test_float(M, N, kb, dt):
    hero, f8 = pkg.load(), dt == torch.float8_e4m3fn
    K, amp, out = kb // dt.itemsize, 60 if f8 else 1, torch.bfloat16 if f8 else dt
    g = torch.Generator(device="cuda").manual_seed(M * 3 + N)
    a = (torch.randn((M, K), device="cuda", generator=g) * amp).to(dt)
    w = (torch.randn((N, K), device="cuda", generator=g) * amp).to(dt)
    bias = torch.randn(N, device="cuda", generator=g) * K ** 0.5
    res = torch.randn((M, N), device="cuda", generator=g).to(out)
    if f8:
        rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / 3600
        y, s = hero.hero_fp8_gemm(a, w, rs, cs, bias, residual=res, epi=HB.EPI_DEQUANT, out_dtype=out), rs.double()[:, None] * cs.double()
    else:
        y, s = hero.hero_hp_gemm(a, w, bias, residual=res), 1.0
    ref = (a.double() @ w.double().t()) * s + bias.double() + res.double()
    # fp32 sums of K products in any order: (K + 4) * 2^-24 of the sum of the magnitudes; then one rounding to the result's type
    bound = (K + 4) * 2.0 ** -24 * ((a.double().abs() @ w.double().abs().t()) * s + bias.double().abs() + res.double().abs())
    ulp = 2.0 ** -8 if out == torch.bfloat16 else 2.0 ** -11
    assert bool(((y.double() - ref).abs() <= bound + (ref.abs() + bound) * ulp).all())


@pytest.mark.gpu
@pytest.mark.parametrize("dt", DTYPES[2:])
@pytest.mark.parametrize("M,N", [(3, 4096), (32, 4112)])
def test_residual_rows_anywhere(M, N, dt):
    """The 16-bit product takes a residual of any row stride and address: the same bits as from aligned rows."""
    hero, K, g = pkg.load(), 512, torch.Generator(device="cuda").manual_seed(M)
    a, w = torch.randn((M, K), device="cuda", generator=g).to(dt), torch.randn((N, K), device="cuda", generator=g).to(dt)
    res = torch.randn((M, N), device="cuda", generator=g).to(dt)
    want = hero.hero_hp_gemm(a, w, residual=res)
    for pad, off in ((1, 0), (3, 1), (4, 1), (4, 2), (2, 3), (0, 1)):
        flat = torch.full((M * (N + pad) + 8,), float("nan"), dtype=dt, device="cuda")
        view = flat[off:off + M * (N + pad)].view(M, N + pad)[:, :N]
        view.copy_(res)
        assert torch.equal(hero.hero_hp_gemm(a, w, residual=view), want), (pad, off)


@pytest.mark.gpu
@pytest.mark.parametrize("d,f,fmt", [(2048, 4160, "i8"), (4096, 16384, "i8"), (2048, 2048, "fp8"), (4096, 4096, "f16")])
def test_fused_ln_quant(d, f, fmt):
    """A pre-LN layer of one token per sequence: with up to eight rows each LN^quant runs inside the linear behind it, with nine it
    does not.  The statistics' sums are ordered differently, nothing else: a row's result is the same but for re-rounded codes."""
    hero = pkg.load()
    H, Dh, fp8 = d // 128, 128, fmt == "fp8"
    mode = HB.MODE_M3 | (HB.M_FP8 if fp8 else HB.M_F16 if fmt == "f16" else 0)
    hp = torch.float16 if fmt == "f16" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(d)
    p = {k: torch.randn(s, device="cuda", generator=g) * 0.03 for k, s in
         {"w_qkv": (d, 3 * d), "b_qkv": (3 * d,), "w_o": (d, d), "b_o": (d,), "w_1": (d, f), "b_1": (f,), "w_2": (f, d), "b_2": (d,)}.items()}
    for k in ("ln1", "ln2"):
        p[k + "_g"], p[k + "_b"] = 1 + 0.1 * torch.randn(d, device="cuda", generator=g), 0.1 * torch.randn(d, device="cuda", generator=g)
    x = torch.randn((2 * 64, d), device="cuda", generator=g).double()
    sc, _ = prep.calibrate(p, x, HB.ARCH_PRE_LN, H, Dh, 1e-5, HB.MASK_CAUSAL, 2, 64, hero=hero, fp8=fp8)
    t, qk, ps = prep.prepare(p, sc, HB.ARCH_PRE_LN, d, Dh, mode & ~HB.M_FP8, hero=hero, fp8=fp8)
    h0 = (torch.randn((9, d), device="cuda", generator=g) * 3 + 0.5).to(hp)
    h0[2] = 0                                                        # a row without variance
    for beta in (True, False):
        if not beta:
            t = {k: v for k, v in t.items() if k not in ("ln1_b", "ln2_b")}
        W, desc = hero.layer_weights(t, qk, ps), hero.layer_desc(HB.ARCH_PRE_LN, d, H, Dh, f, 1e-5, HB.MASK_CAUSAL, mode)

        def run(h):
            n = h.shape[0]
            ws = torch.full((hero.hero_layer_workspace_bytes(desc, n, 1),), 0xA5, dtype=torch.uint8, device="cuda")
            kc = torch.zeros((n, H, 4, Dh), dtype=torch.float8_e4m3fn if fp8 else torch.int8, device="cuda")
            vc, out = torch.zeros_like(kc), h.clone()
            hero.hero_layer_fwd(desc, W, n, 1, ws, h=out, kv_len=torch.ones(n, dtype=torch.int32, device="cuda"), k_cache=kc, v_cache=vc)
            return out, kc[:, :, 0], vc[:, :, 0]
        nine = run(h0)
        for M in (1, 3, 8):
            few = run(h0[:M])
            assert bool(torch.isfinite(few[0].float()).all())
            for q, r in zip(few[1:], nine[1:]):                      # the appended K / V codes: behind one LN^quant
                assert float((q.float() != r[:M].float()).float().mean()) <= 1e-3
            assert float((few[0].float() - nine[0][:M].float()).norm() / nine[0][:M].float().norm()) <= 2e-3
