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


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,kb", SHAPES)
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float8_e4m3fn])
def test_floats(M, N, kb, dt, tile):
    if dt == torch.float8_e4m3fn and tile in (10, 12):
        pytest.skip("E4M3 has tiles of 256, 192 and 128 rows")
    hero, K = pkg.load(), kb // dt.itemsize
    a, w, rs, cs, bias, _ = _inputs(M, N, K, dt)
    ref, mag = a.double() @ w.double().t(), a.double().abs() @ w.double().abs().t()
    if dt == torch.bfloat16:
        y, ref = hero.hero_hp_gemm(a, w, bias, tile=tile), ref + bias.double()
        bound = (K + 4) * 2.0 ** -24 * (mag + bias.double().abs())                  # fp32 sums in any order
    else:
        y, s = hero.hero_fp8_gemm(a, w, rs, cs, bias, tile=tile, out_dtype=torch.bfloat16), rs.double()[:, None] * cs.double()
        ref = ref * s + bias.double()
        bound = (2.0 ** -12 + (K + 4) * 2.0 ** -24) * (mag * s + bias.double().abs())     # products kept to 13 bits of the largest of eight
    assert bool(((y.double() - ref).abs() <= bound + (ref.abs() + bound) * 2.0 ** -8).all())
