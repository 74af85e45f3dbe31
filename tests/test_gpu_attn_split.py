"""The two INT8 / E4M3 attention kernels against each other: the same sequences alone (the keys split over a block's waves) and
repeated until the launch has more than one 128-query block per CU (the 128-query kernel).  Both follow the oracle's
formulas; they add a row's exponentials in another order, so a probability or an output code may part at a rounding tie."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("Sq,Skv", [(33, 33), (64, 64), (129, 129), (150, 150), (40, 300), (97, 261), (513, 513)])
def test_split_against_block(Dh, fp8, mask, Sq, Skv):
    if mask == HB.MASK_CAUSAL or Sq == Skv:
        lens = [Skv, Skv - 1, max(1, Skv // 2), 1 if mask == HB.MASK_PADDING else Skv]
    else:
        lens = [Skv, Skv // 2, 31, 1]
    hero, B, H = pkg.load(), 4, 3
    g = torch.Generator(device="cuda").manual_seed(Sq + Skv)
    dt = torch.float8_e4m3fn if fp8 else torch.int8
    draw = lambda S: (torch.randn((B, S, H, Dh), device="cuda", generator=g) * (60 if fp8 else 30)).clamp(-127, 127).to(dt)
    q, k, v = draw(Sq), draw(Skv), draw(Skv)
    kv = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ps = 1 / 448 if fp8 else 1 / 255
    scale = torch.rand(H * Dh, device="cuda", generator=g) * ps + ps / 2
    fn = hero.hero_fp8_attn if fp8 else hero.hero_int8_attn
    call = lambda r: fn(*(t.repeat(r, 1, 1, 1) for t in (q, k, v)), 0.02 / Dh ** 0.5 / (4 if fp8 else 1), ps, scale,
                        mask=mask, kv_len=kv.repeat(r))
    reps = 256 // (B * H * ((Sq + 127) // 128)) + 1
    one, many = call(1), call(reps)
    many = many.view(torch.int8).view(reps, B * Sq, H * Dh)
    assert torch.equal(many, many[:1].expand_as(many))
    a, b = one.view(torch.int8), many[0]
    # a probability in code units is good to some 255 * 4 * 2^-24 = 6e-5 (its sum of exponentials is ordered otherwise), so
    # about one code in 2e4 may part (E4M3 has a quarter of the ties per step but also rounds the output), and each moves at
    # most the Dh outputs of its row by one code
    assert int((a != b).sum()) <= (5e-5 * B * H * Sq * Skv + 3) * Dh
    if fp8:
        x, y = one.float(), b.view(dt).float()
        assert float((x - y).abs().max()) <= 2.0 ** -3 * float(x.abs().max())
    else:
        assert int((a.int() - b.int()).abs().max()) <= 1


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("Sq,Skv", [(1, 1), (20, 77), (33, 33), (129, 129), (97, 261), (513, 513)])
def test_16_bit_split_against_block(Dh, dt, mask, Sq, Skv):
    """The 16-bit attention likewise, and both against 64 bits: the probabilities are rounded to 16 bits before PV (relative
    2^-9 for bf16, 2^-12 for fp16), the output once more."""
    lens = [Skv, Skv - 1 if Sq < Skv or mask == HB.MASK_PADDING else Skv, max(1, Skv // 2) if Sq == Skv and mask != HB.MASK_CAUSAL else Skv]
    hero, B, H = pkg.load(), 3, 3
    g = torch.Generator(device="cuda").manual_seed(Sq + Skv)
    q, k, v = (torch.randn((B, s, H, Dh), device="cuda", generator=g).to(dt) for s in (Sq, Skv, Skv))
    kv = torch.tensor(lens, dtype=torch.int32, device="cuda")
    scale = 2.0 / Dh ** 0.5
    call = lambda r: hero.hero_hp_attn(*(t.repeat(r, 1, 1, 1) for t in (q, k, v)), scale, mask=mask, kv_len=kv.repeat(r))
    outs = [call(1)]
    if Sq > 32:
        outs.append(call(256 // (B * H * ((Sq + 127) // 128)) + 1)[:B * Sq])
    a = torch.einsum("bihd,bjhd->bhij", q.double().cpu(), k.double().cpu()) * scale
    i, j, n = torch.arange(Sq)[:, None], torch.arange(Skv)[None, :], kv.cpu()[:, None, None]
    vis = (j < n) & ((j <= i + n - Sq) if mask == HB.MASK_CAUSAL else torch.ones_like(n, dtype=torch.bool))
    if mask == HB.MASK_PADDING and Sq == Skv:
        vis = vis & (i < n)
    p = torch.softmax(a.masked_fill(~vis[:, None], -1e300), 3) * vis[:, None]
    ref = torch.einsum("bhij,bjhd->bihd", p, v.double().cpu()).reshape(B * Sq, H * Dh)
    mag = torch.einsum("bhij,bjhd->bihd", p, v.double().cpu().abs()).reshape(B * Sq, H * Dh)
    eps = 2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -11
    for o in outs:
        assert bool(((o.double().cpu() - ref).abs() <= 2 * eps * mag + eps * ref.abs() + 1e-6).all())
