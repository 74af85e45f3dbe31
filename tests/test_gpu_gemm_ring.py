"""The direct-to-LDS ring GEMM (small and middling problems): every form of its rule at the edges of its tiles, against the
same product in 64 bits.  Shapes: one row / one column past a tile, ragged N, K of one slab, K that the K groups share
unevenly (empty groups among them), K that ends in half a slab.  test_gemm_routes.py checks that they reach every form."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB, prep

pytestmark = pytest.mark.gpu

# M, N, K in bytes of the operands; the comment names the form that the rule picks
SHAPES = [
    (1, 32, 128),            # 32x32, one slab for eight groups
    (33, 100, 896),          # 32x32, seven slabs over eight groups
    (7, 4000, 8192 + 128),   # 32x32, four groups, 65 slabs
    (31, 12284, 2176),       # 32x64, two groups, 17 slabs
    (32, 12300, 8192),       # 32x64, four groups
    (65, 2308, 640),         # 32x32, five slabs over eight groups, three row tiles
    (65, 3076, 640),         # 64x32, four groups
    (100, 4092, 4224),       # 64x32, four groups, 33 slabs
    (127, 3000, 128),        # 64x32, one slab for four groups
    (651, 764, 3072),        # 32x64, four groups, many row tiles
    (129, 4612, 768),        # 64x64, two groups
    (100, 12292, 4224),      # 128x64, two groups, 33 slabs
    (641, 2052, 384),        # 64x64
    (300, 10244, 4096),      # 128x128
    (1025, 2300, 1024),      # 128x64
    (65, 260, 192),          # 32x32, one and a half slabs
    # few rows of many columns
    (3, 36868, 4096),        # 32x64, two groups, more tiles than a round
    (64, 33004, 1024),       # 64x64
    # K that ends in half a slab, in every form
    (1, 32, 64),             # 32x32, half a slab for eight groups
    (33, 100, 832),          # 32x32, eight groups
    (7, 4000, 8256),         # 32x32, four groups
    (31, 12284, 2112),       # 32x64, two groups
    (32, 12300, 8256),       # 32x64, four groups
    (100, 4092, 4160),       # 64x32, four groups
    (129, 4612, 832),        # 64x64, two groups
    (100, 12292, 4160),      # 128x64, two groups
    (641, 2052, 320),        # 64x64
    (1025, 2300, 960),       # 128x64
    (1100, 4100, 4160),      # 128x128, more tiles than a round
    (1500, 4100, 1088),      # (the register-staged kernel: K too short for that)
]


def _strided(t, extra):
    """The same matrix inside rows that are `extra` elements longer."""
    buf = torch.zeros((t.shape[0], t.shape[1] + extra), dtype=t.dtype, device=t.device)
    buf[:, :t.shape[1]] = t
    return buf[:, :t.shape[1]]


@pytest.mark.parametrize("M,N,kb", SHAPES)
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("gelu,res", [(False, False), (False, True), (True, False), (True, True)])
def test_hp_gemm_forms(M, N, kb, dt, gelu, res):
    hero, K = pkg.load(), kb // 2
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N)
    a = _strided(torch.randn((M, K), device="cuda", generator=g).to(dt), 8)
    w = (torch.randn((N, K), device="cuda", generator=g) * K ** -0.5).to(dt)
    bias = torch.randn(N, device="cuda", generator=g)
    r = _strided(torch.randn((M, N), device="cuda", generator=g).to(dt), 4) if res else None
    y = hero.hero_hp_gemm(a, w, bias, residual=r, gelu=gelu)
    ref = a.double() @ w.double().t() + bias.double()
    # fp32 sums of K products in any order: K * 2^-24 of the sum of the magnitudes; GELU's slope is below 1.13
    bound = 1.13 * (K + 2) * 2.0 ** -24 * (a.double().abs() @ w.double().abs().t() + bias.double().abs())
    if gelu:
        ref = torch.nn.functional.gelu(ref)
        bound = bound + 2.0 ** -22
    if res:
        ref = ref + r.double()
    ulp = 2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -11        # half a unit in the last place
    assert bool(((y.double() - ref).abs() <= bound + (ref.abs() + bound) * ulp + 2.0 ** -25).all())


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_int8_gemm_forms(M, N, K):
    """Integer sums are exact in any order: the raw product, and one rounding behind the pinned epilogue."""
    hero = pkg.load()
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a = _strided(torch.randint(-127, 128, (M, K), device="cuda", generator=g, dtype=torch.int8), 16)
    w = torch.randint(-127, 128, (N, K), device="cuda", generator=g, dtype=torch.int8)
    acc = (a.double() @ w.double().t()).to(torch.int32)
    assert torch.equal(hero.hero_int8_gemm(a, w), acc)
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / (90 * K ** 0.5)
    bias = torch.randn(N, device="cuda", generator=g)
    res = torch.randn((M, N), device="cuda", generator=g).to(torch.bfloat16)
    x = acc.float() * rs[:, None]                                    # one fp32 product, then one fused multiply-add
    y = (x.double() * cs.double() + bias.double()).float()
    got = hero.hero_int8_gemm(a, w, rs, cs, bias, residual=res, epi=HB.EPI_DEQUANT, out_dtype=torch.bfloat16)
    # (the double sum is rounded twice, the fused instruction once: they part at most at a tie, one code in some millions)
    assert float((got != (y + res.float()).to(torch.bfloat16)).float().mean()) <= 1e-6
    got = hero.hero_int8_gemm(a, w, rs, cs * 40, bias * 40, epi=HB.EPI_REQUANT, out_dtype=torch.int8)
    y = (x.double() * (cs * 40).double() + (bias * 40).double()).float()
    assert int((got.int() - y.round().clamp(-127, 127).int()).abs().max()) <= 1
    assert float((got.int() != y.round().clamp(-127, 127).int()).float().mean()) <= 1e-6


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_fp8_gemm_forms(M, N, K):
    hero = pkg.load()
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a = (torch.randn((M, K), device="cuda", generator=g) * 60).clamp(-448, 448).to(torch.float8_e4m3fn)
    w = (torch.randn((N, K), device="cuda", generator=g) * 60).clamp(-448, 448).to(torch.float8_e4m3fn)
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / (3600 * K ** 0.5)
    bias = torch.randn(N, device="cuda", generator=g)
    y = hero.hero_fp8_gemm(a, w, rs, cs, bias, epi=HB.EPI_DEQUANT, out_dtype=torch.bfloat16)
    s = rs.double()[:, None] * cs.double()
    ref = (a.double() @ w.double().t()) * s + bias.double()
    # fp32 sums in any order: (K + 4) * 2^-24 of the sum of the magnitudes; then one rounding to bf16
    bound = (K + 4) * 2.0 ** -24 * ((a.double().abs() @ w.double().abs().t()) * s + bias.double().abs())
    assert bool(((y.double() - ref).abs() <= bound + (ref.abs() + bound) * 2.0 ** -8).all())


@pytest.mark.parametrize("M", [1, 33, 64, 100])
def test_int8_split_half_slab(M):
    """The K split of a skinny product whose K ends in half a slab: raw sums exact, through a scratch that is dirty."""
    hero, N, K = pkg.load(), 1028, 8192 + 64
    g = torch.Generator(device="cuda").manual_seed(M)
    a = _strided(torch.randint(-127, 128, (M, K), device="cuda", generator=g, dtype=torch.int8), 16)
    w = torch.randint(-127, 128, (N, K), device="cuda", generator=g, dtype=torch.int8)
    ws = torch.full((hero.hero_int8_gemm_workspace_bytes(M, N, K),), 0xA5, dtype=torch.uint8, device="cuda")
    assert ws.numel() > 0
    assert torch.equal(hero.hero_int8_gemm(a, w, workspace=ws), (a.double() @ w.double().t()).to(torch.int32))


@pytest.mark.parametrize("B,fmt,f", [(b, t, 8192) for b in (1, 5, 64, 100) for t in ("fp8", "bf16")] +
                         [(129, "bf16", 16384 + 64), (300, "bf16", 16384), (700, "bf16", 16384)])
def test_layer_split_k(B, fmt, f):
    """One token per sequence through a layer whose FC2 is long enough for the K split (E4M3 codes, or 16 bits: skinny, and
    middling with 128 x 256 tiles), through a scratch that is dirty, against the same again and against single rows."""
    hero = pkg.load()
    d, H, Dh = 1024, 8, 128
    mode = HB.MODE_M3 | HB.M_FP8 if fmt == "fp8" else HB.MODE_M2
    g = torch.Generator(device="cuda").manual_seed(B)
    p = {k: torch.randn(s, device="cuda", generator=g) * 0.03 for k, s in
         {"w_qkv": (d, 3 * d), "b_qkv": (3 * d,), "w_o": (d, d), "b_o": (d,), "w_1": (d, f), "b_1": (f,), "w_2": (f, d), "b_2": (d,)}.items()}
    for k in ("ln1", "ln2"):
        p[k + "_g"], p[k + "_b"] = 1 + 0.1 * torch.randn(d, device="cuda", generator=g), torch.zeros(d, device="cuda")
    x = torch.randn((2 * 64, d), device="cuda", generator=g).double()
    sc, _ = prep.calibrate(p, x, HB.ARCH_PRE_LN, H, Dh, 1e-5, HB.MASK_CAUSAL, 2, 64, hero=hero, fp8=fmt == "fp8")
    t, qk, ps = prep.prepare(p, sc, HB.ARCH_PRE_LN, d, Dh, mode & ~HB.M_FP8, hero=hero, fp8=fmt == "fp8")
    W, desc = hero.layer_weights(t, qk, ps), hero.layer_desc(HB.ARCH_PRE_LN, d, H, Dh, f, 1e-5, HB.MASK_CAUSAL, mode)
    h0 = torch.randn((B, d), device="cuda", generator=g).to(torch.bfloat16)

    def run(h, poison):
        n = h.shape[0]
        ws = torch.full((hero.hero_layer_workspace_bytes(desc, n, 1),), poison, dtype=torch.uint8, device="cuda")
        kc = torch.zeros((n, H, 4, Dh), dtype=torch.float8_e4m3fn if fmt == "fp8" else torch.int8, device="cuda")
        vc, out = torch.zeros_like(kc), h.clone()
        hero.hero_layer_fwd(desc, W, n, 1, ws, h=out, kv_len=torch.ones(n, dtype=torch.int32, device="cuda"), k_cache=kc, v_cache=vc)
        return out
    one = run(h0, 0xFF)
    assert bool(torch.isfinite(one.float()).all())
    assert torch.equal(one, run(h0, 0x00))
    # every row on its own is in the same class (another form may serve it: the fp32 sums are ordered otherwise)
    rows = torch.cat([run(h0[b:b + 1], 0xFF) for b in range(0, B, max(1, B // 3))]).float()
    sel = one[0:B:max(1, B // 3)].float()
    assert float((rows - sel).norm() / sel.norm()) <= 1e-2
