"""The direct-to-LDS ring GEMM (small and middling problems): every form of its rule at the edges of its tiles, against the
same product in 64 bits.  Shapes: one row / one column past a tile, ragged N, K of one slab, K that the K groups share
unevenly (empty groups among them), K that is no whole slab (the register-staged kernel)."""
import pytest
import torch

import paper_2310_17723_amd as pkg

pytestmark = pytest.mark.gpu

# M, N, K in bytes of the operands; the comment names the form that the rule picks
SHAPES = [
    (1, 32, 128),            # 32x32, one slab for eight groups
    (33, 100, 896),          # 32x32, seven slabs over eight groups
    (7, 4000, 8192 + 128),   # 32x32, four groups, 65 slabs
    (31, 12284, 2176),       # 32x64, two groups, 17 slabs
    (32, 12300, 8192),       # 32x64, four groups
    (65, 2308, 640),         # 64x32
    (129, 3076, 768),        # 64x64, two groups
    (100, 12292, 4224),      # 128x64, two groups, 33 slabs
    (641, 2052, 384),        # 64x64
    (300, 10244, 4096),      # 128x128
    (1025, 2300, 1024),      # 128x64
    (65, 260, 192),          # K is one and a half slabs
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
