"""The persistent GEMM's 16 x 16 tiles: a lane's 16 columns cut off by N at every place, rows by M, strides that are and are not multiples
of 16 bytes, both tile sizes and every epilogue, against the ring kernel (INT8: the same bits) and 64 bits (16-bit operands); nothing is
written beside or behind the result."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB

pytestmark = pytest.mark.gpu
SHAPES = [(2049, 2048 + n, 256) for n in range(1, 16)] + [(2049, 2116, 256), (1793, 2304, 1024), (2048, 2176, 384)]


def _canvas(M, N, dtype, step):
    """M rows of N elements whose stride is a multiple of `step` elements (more than N), a row behind them, and what is beside them filled."""
    buf = torch.full((M + 1, (N // step + 1) * step), 3, dtype=dtype, device="cuda")
    return buf, buf[:M, :N]


def _untouched(buf, M, N):
    return bool((buf[:, N:] == 3).all()) and bool((buf[M:] == 3).all())


@pytest.mark.parametrize("tile", [7, 8])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_int8(M, N, K, tile):
    hero = pkg.load()
    g = torch.Generator(device="cuda").manual_seed(N + K)
    a, w = (torch.randint(-127, 128, (n, K), device="cuda", generator=g, dtype=torch.int8) for n in (M, N))
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / (90 * K ** 0.5)
    bias, S = torch.randn(N, device="cuda", generator=g), torch.rand(N, device="cuda", generator=g) / 30 + 0.02
    res = _canvas(M, N, torch.bfloat16, 4)[1]
    res.copy_(torch.randn((M, N), device="cuda", generator=g))
    scaled = dict(a_row_scale=rs, b_col_scale=cs, bias=bias)
    for e in (dict(epi=HB.EPI_RAW_I32, dt=torch.int32), dict(epi=HB.EPI_REQUANT, dt=torch.int8, **scaled),
              dict(epi=HB.EPI_GELU_REQUANT, dt=torch.int8, out_col_scale=S, **scaled), dict(epi=HB.EPI_DEQUANT, dt=torch.float16, **scaled),
              dict(epi=HB.EPI_DEQUANT_GELU, dt=torch.bfloat16, **scaled), dict(epi=HB.EPI_DEQUANT, dt=torch.bfloat16, residual=res, **scaled)):
        dt = e.pop("dt")
        for step in (4, 16):
            (buf, out), (_, other) = _canvas(M, N, dt, step), _canvas(M, N, dt, step)
            hero.hero_int8_gemm(a, w, C_out=out, tile=tile, **e)
            hero.hero_int8_gemm(a, w, C_out=other, tile=2, **e)
            assert torch.equal(out, other) and _untouched(buf, M, N), (e["epi"], step)


@pytest.mark.parametrize("tile", [7, 8])
@pytest.mark.parametrize("M,N,kb", SHAPES)
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
def test_16_bits(M, N, kb, dt, tile):
    hero, K = pkg.load(), kb // 2
    g = torch.Generator(device="cuda").manual_seed(N + K)
    a, w = torch.randn((M, K), device="cuda", generator=g).to(dt), (torch.randn((N, K), device="cuda", generator=g) * K ** -0.5).to(dt)
    bias, res = torch.randn(N, device="cuda", generator=g), torch.randn((M, N), device="cuda", generator=g).to(dt)
    ref = a.double() @ w.double().t() + bias.double() + res.double()
    # fp32 sums of K products in any order: (K + 4) * 2^-24 of the sum of the magnitudes; then one rounding
    bound = (K + 4) * 2.0 ** -24 * (a.double().abs() @ w.double().abs().t() + bias.double().abs() + res.double().abs())
    ulp = 2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -11
    for step, rows in ((4, res), (8, _canvas(M, N, dt, 1)[1])):      # the residual's rows on wide boundaries and on odd ones
        rows.copy_(res)
        buf, y = _canvas(M, N, dt, step)
        hero.hero_hp_gemm(a, w, bias, residual=rows, C_out=y, tile=tile)
        assert bool(((y.double() - ref).abs() <= bound + (ref.abs() + bound) * ulp).all()) and _untouched(buf, M, N), step


@pytest.mark.parametrize("tile", [7, 8, 10, 11, 12])
@pytest.mark.parametrize("M,N", [(2048, 2304), (2047, 2304), (2049, 2303), (1793, 2312)])
def test_16_bit_results_whole_and_cut_tiles(M, N, tile):
    """Tiles whose rows all exist take a path of their own, without a row scale and bias as with them: the ring kernel's bits."""
    hero, K = pkg.load(), 384
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = (torch.randint(-127, 128, (n, K), device="cuda", generator=g, dtype=torch.int8) for n in (M, N))
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / (90 * K ** 0.5)
    for dt in (torch.float16, torch.bfloat16):
        for epi in (HB.EPI_DEQUANT, HB.EPI_DEQUANT_GELU):
            for kw in (dict(a_row_scale=rs, bias=cs * 30), dict()):
                for step in (4, 8):
                    (buf, out), (_, other) = _canvas(M, N, dt, step), _canvas(M, N, dt, step)
                    hero.hero_int8_gemm(a, w, b_col_scale=cs, epi=epi, C_out=out, tile=tile, **kw)
                    hero.hero_int8_gemm(a, w, b_col_scale=cs, epi=epi, C_out=other, tile=2, **kw)
                    assert torch.equal(out, other) and _untouched(buf, M, N), (dt, epi, bool(kw), step)


@pytest.mark.parametrize("tile", [7, 8, 10, 11, 12])
@pytest.mark.parametrize("M,N", [(2049, 2312), (1793, 2307), (300, 2305)])
def test_residual_off_wide_boundaries(M, N, tile):
    """Pieces whose 16 columns all exist, and ones that N cuts, of a residual that lies on 2, 4 and 8 bytes: the bits of one that lies on 16, and
    (INT8) those of the ring kernel."""
    hero, K = pkg.load(), 384
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = (torch.randint(-127, 128, (n, K), device="cuda", generator=g, dtype=torch.int8) for n in (M, N))
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / (90 * K ** 0.5)
    bias, r = torch.randn(N, device="cuda", generator=g), torch.randn((M, N), device="cuda", generator=g)
    for dt in (torch.float16, torch.bfloat16):
        x, y = torch.randn((M, K), device="cuda", generator=g).to(dt), (torch.randn((N, K), device="cuda", generator=g) * K ** -0.5).to(dt)
        first = {}
        for ldr, off in ((2320, 0), (2324, 0), (2320, 1), (2320, 4), (2321, 0), (2322, 2)):
            res = torch.full((M * ldr + off,), 9, dtype=dt, device="cuda")[off:].view(M, ldr)[:, :N]
            res.copy_(r)
            calls = {"linear": lambda c: hero.hero_hp_gemm(x, y, bias, residual=res, C_out=c, tile=tile),
                     "gelu": lambda c: hero.hero_hp_gemm(x, y, bias, residual=res, gelu=True, C_out=c, tile=tile)}
            if ldr % 4 == 0 and off == 0:                                # all that 8-bit operands come with
                calls["i8"] = lambda c: hero.hero_int8_gemm(a, w, rs, cs, bias, residual=res, epi=HB.EPI_DEQUANT, C_out=c, tile=tile)
            for name, call in calls.items():
                buf, out = _canvas(M, N, dt, 16)
                call(out)
                assert torch.equal(first.setdefault(name, out), out) and _untouched(buf, M, N), (dt, name, ldr, off)
            if "i8" in calls:
                _, other = _canvas(M, N, dt, 16)
                hero.hero_int8_gemm(a, w, rs, cs, bias, residual=res, epi=HB.EPI_DEQUANT, C_out=other, tile=2)
                assert torch.equal(first["i8"], other), (dt, ldr, off)


@pytest.mark.parametrize("M,N,K", [(8065, 8200, 4096), (7937, 8448, 4224), (16384, 4097, 4096)])
def test_the_branch_free_loop(M, N, K):
    """1024 tiles of 256 x 256 and more, each of 64 slabs or more (66: the activations' ring of four slots starts the next tile at another one): the
    last iterations of a tile are code of their own there.  INT8 against the ring kernel's bits, 16 bits against 64 on rows of several tiles."""
    assert -(-M // 256) * -(-N // 256) >= 1024 and K >= 64 * 64      # what launch_persistent_tile asks for
    hero = pkg.load()
    g = torch.Generator(device="cuda").manual_seed(M + K)
    a, w = (torch.randint(-127, 128, (n, K), device="cuda", generator=g, dtype=torch.int8) for n in (M, N))
    rs, cs = torch.rand(M, device="cuda", generator=g) + 0.5, (torch.rand(N, device="cuda", generator=g) + 0.5) / (90 * K ** 0.5)
    bias, res = torch.randn(N, device="cuda", generator=g), {}
    for dt in (torch.bfloat16, torch.float16):
        res[dt] = _canvas(M, N, dt, 16)[1]
        res[dt].copy_(torch.randn((M, N), device="cuda", generator=g))
    scaled = dict(a_row_scale=rs, b_col_scale=cs, bias=bias)
    kinds = [dict(epi=HB.EPI_RAW_I32, dt=torch.int32), dict(epi=HB.EPI_REQUANT, dt=torch.int8, **scaled)]
    for dt in res:
        kinds += [dict(epi=HB.EPI_DEQUANT, dt=dt, **scaled), dict(epi=HB.EPI_DEQUANT_GELU, dt=dt, **scaled), dict(epi=HB.EPI_DEQUANT, dt=dt, residual=res[dt], **scaled)]
    for e in kinds:
        dt = e.pop("dt")
        (buf, out), (_, other) = _canvas(M, N, dt, 16), _canvas(M, N, dt, 16)
        hero.hero_int8_gemm(a, w, C_out=out, tile=7, **e)
        hero.hero_int8_gemm(a, w, C_out=other, tile=2, **e)
        assert torch.equal(out, other) and _untouched(buf, M, N), (e["epi"], dt, "residual" in e)
    rows = torch.tensor([0, 255, 256, M // 2, M - 257, M - 1], device="cuda")
    for dt, ulp in ((torch.bfloat16, 2.0 ** -8), (torch.float16, 2.0 ** -11)):
        x, y = torch.randn((M, K // 2), device="cuda", generator=g).to(dt), (torch.randn((N, K // 2), device="cuda", generator=g) * K ** -0.5).to(dt)
        xs, rr = x[rows].double(), res[dt][rows].double()
        lin = xs @ y.double().t() + bias.double()
        sums = (K + 4) * 2.0 ** -24 * (xs.abs() @ y.double().abs().t() + bias.double().abs())
        for gelu in (False, True):
            for r in (None, res[dt]):
                buf, out = _canvas(M, N, dt, 8)
                hero.hero_hp_gemm(x, y, bias, residual=r, gelu=gelu, C_out=out, tile=7)      # half of K: the same slabs of 16 bits
                act = torch.nn.functional.gelu(lin) if gelu else lin
                ref = act + (rr if r is not None else 0)
                # GELU's slope is at most 1.13, its fp32 form within 1.1e-7 and a rounding; the residual's sum rounds once
                bound = (1.13 * sums + 1.1e-7 + 2.0 ** -24 * act.abs() if gelu else sums) + (2.0 ** -24 * ref.abs() if r is not None else 0)
                assert bool(((out[rows].double() - ref).abs() <= bound + (ref.abs() + bound) * ulp).all()) and _untouched(buf, M, N), (dt, gelu, r is not None)
