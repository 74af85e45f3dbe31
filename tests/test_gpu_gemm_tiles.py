"""The persistent GEMM where a workgroup walks several tiles: its two rings and the epilogue's vectors pass from tile to tile, from the shortest K
it takes (two pairs of slabs) on; every height of its tiles, whose last loads are for a part of the waves only."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB

pytestmark = pytest.mark.gpu
TILES = [7, 8, 10, 11, 12]
SHAPES = [(4500, 4200, kb) for kb in (256, 384, 512, 640)] + [(4500, 4208, 1024)]      # 306 tiles of 256 x 256, 1188 of 128 x 128
# rows in front of, at and behind the edges of a tile, of a wave's half and of a load's 16 rows
SHAPES += [(n, 2304, 512) for n in (1, 16, 79, 80, 81, 160, 161, 191, 193, 223, 225, 273)]


def _inputs(M, N, K, dt):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    if dt == torch.int8:
        a, w = (torch.randint(-127, 128, (n, K), device="cuda", generator=g, dtype=torch.int8) for n in (M, N))
    else:
        a, w = (torch.randn((n, K), device="cuda", generator=g).to(dt) for n in (M, N))
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, torch.rand(N, device="cuda", generator=g) + 0.5
    return a, w, rs, cs, torch.randn(N, device="cuda", generator=g), torch.rand(N, device="cuda", generator=g) / 30 + 0.02


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_int8(M, N, K, tile):
    hero = pkg.load()
    a, w, rs, cs, bias, S = _inputs(M, N, K, torch.int8)
    cs = cs / (90 * K ** 0.5)
    for epi, kw in ((HB.EPI_REQUANT, {}), (HB.EPI_GELU_REQUANT, {"out_col_scale": S})):
        out, ring = (hero.hero_int8_gemm(a, w, rs, cs, bias, epi=epi, out_dtype=torch.int8, tile=t, **kw) for t in (tile, 2))
        assert torch.equal(out, ring), epi
    assert torch.equal(hero.hero_int8_gemm(a, w, tile=tile), hero.hero_int8_gemm(a, w, tile=2))


@pytest.mark.parametrize("M,N,kb", SHAPES)
@pytest.mark.parametrize("dt,tile", [(dt, t) for dt in (torch.bfloat16, torch.float16) for t in TILES] + [(torch.float8_e4m3fn, t) for t in (7, 8, 11)])
def test_floats(M, N, kb, dt, tile):
    hero, K = pkg.load(), kb // dt.itemsize
    a, w, rs, cs, bias, _ = _inputs(M, N, K, dt)
    ref, mag = a.double() @ w.double().t(), a.double().abs() @ w.double().abs().t()
    if dt != torch.float8_e4m3fn:
        y, ref = hero.hero_hp_gemm(a, w, bias, tile=tile), ref + bias.double()
        bound = (K + 4) * 2.0 ** -24 * (mag + bias.double().abs())                  # fp32 sums in any order
    else:
        y, s = hero.hero_fp8_gemm(a, w, rs, cs, bias, tile=tile, out_dtype=torch.bfloat16), rs.double()[:, None] * cs.double()
        ref = ref * s + bias.double()
        bound = (2.0 ** -12 + (K + 4) * 2.0 ** -24) * (mag * s + bias.double().abs())     # products kept to 13 bits of the largest of eight
    assert bool(((y.double() - ref).abs() <= bound + (ref.abs() + bound) * (2.0 ** -11 if dt == torch.float16 else 2.0 ** -8)).all())


@pytest.mark.parametrize("M,N,K", [(1100, 4096, 16384), (1053, 4100, 16512), (602, 4096, 16384)])
def test_a_buffer_the_size_query_does_not_ask_for_stays_as_it_is(M, N, K):
    """hero_int8_gemm_workspace_bytes is 0: "any buffer, or none, is accepted", and none is written, also where the layer would split K."""
    hero = pkg.load()
    assert hero.lib.hero_int8_gemm_workspace_bytes(M, N, K) == 0
    a, w, rs, cs, bias, _ = _inputs(M, N, K, torch.int8)
    kw = dict(a_row_scale=rs, b_col_scale=cs / (90 * K ** 0.5), bias=bias, epi=HB.EPI_REQUANT, out_dtype=torch.int8)
    ws = torch.full((8 * M * N * 4,), 0xA5, dtype=torch.uint8, device="cuda")
    assert torch.equal(hero.hero_int8_gemm(a, w, workspace=ws, **kw), hero.hero_int8_gemm(a, w, **kw))
    assert torch.equal(hero.hero_int8_gemm(a, w, workspace=ws), hero.hero_int8_gemm(a, w))
    assert bool((ws == 0xA5).all())


@pytest.mark.parametrize("B,S,f", [(2, 550, 16384), (1, 1053, 16512)])
def test_int8_k_split_of_a_middling_product(B, S, f, monkeypatch):
    """A chunk's FC2 in INT8, two K ranges in tiles of 160 rows (the second one shorter): the sums are exact, so the layer's result is the same bit for bit
    through scratch that is dirty and no larger than it has to be, and without it."""
    import test_gpu_workspace as TW
    monkeypatch.setattr(TW, "D", 4096)
    monkeypatch.setattr(TW, "H", 32)
    hero, mode, T = pkg.load(), HB.MODE_M3, B * S
    keep, W, desc = TW._layer(hero, mode, f, 5)
    full, planes = hero.hero_layer_workspace_bytes(desc, B, S), 2 * T * 4096 * 4
    h0 = torch.randn((T, 4096), device="cuda", generator=torch.Generator(device="cuda").manual_seed(6)).to(torch.bfloat16)
    res = []
    for nbytes in (full, full - planes):
        h, ws = h0.clone(), torch.full((nbytes + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        hero.hero_layer_fwd(desc, W, B, S, ws[:nbytes], h=h)
        res.append(h)
        assert bool((ws[nbytes:] == 0xA5).all())
        if nbytes == full:
            assert not bool((ws[full - planes:full - planes + 4096] == 0xA5).all())
    assert torch.equal(res[0], res[1]) and bool(torch.isfinite(res[0].float()).all())


@pytest.mark.parametrize("mode", [HB.MODE_M2, HB.MODE_M2 | HB.M_F16])
def test_16_bit_k_split_of_a_middling_product(mode, monkeypatch):
    """A chunk's FC2 in 16 bits, split where the workspace has room: the sums part by their fp32 order, a rounding at most behind them."""
    import test_gpu_workspace as TW
    monkeypatch.setattr(TW, "D", 4096)
    monkeypatch.setattr(TW, "H", 32)
    hero = pkg.load()
    keep, W, desc = TW._layer(hero, mode, 8192, 5)
    dt = torch.float16 if mode & HB.M_F16 else torch.bfloat16
    keep["w_2_bf16"] = keep["w_2_bf16"].to(dt)
    W = hero.layer_weights(keep, 2e-4, 1 / 255)
    B, S = 2, 550
    full = hero.hero_layer_workspace_bytes(desc, B, S)
    h0 = torch.randn((B * S, 4096), device="cuda", generator=torch.Generator(device="cuda").manual_seed(6)).to(dt)
    res = []
    for nbytes in (full, full - 2 * B * S * 4096 * 4):               # two planes
        h, ws = h0.clone(), torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        hero.hero_layer_fwd(desc, W, B, S, ws, h=h)
        res.append(h.float())
    assert bool(torch.isfinite(res[0]).all())
    assert float((res[0] - res[1]).norm() / res[0].norm()) <= 2.0 ** -8
