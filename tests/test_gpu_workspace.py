"""What hero_layer_fwd accepts as a workspace: the activations and INT8's split scratch are needed; the split scratch of E4M3 and
16-bit linears is used if it is there."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB

pytestmark = pytest.mark.gpu

D, H, DH = 1024, 8, 128


def _layer(hero, mode, f, seed):
    """A PRE_LN layer of random codes: scales as a calibrated one has them."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float8_e4m3fn if mode & HB.M_FP8 else torch.int8
    codes = lambda *s: (torch.randn(s, device="cuda", generator=g) * 35).clamp(-127, 127).to(dt)
    near = lambda n, s: (torch.rand(n, device="cuda", generator=g) + 0.5) * s
    t = {}
    for w, n, k, s in (("w_qkv", 3 * D, D, 30.0), ("w_o", D, D, 0.5), ("w_1", f, D, 1.0), ("w_2", D, f, 0.5)):
        t[w], t[w + "_s"], t["b_" + w[2:]] = codes(n, k), near(n, s / (35 * k ** 0.5)), near(n, 0.01)
    for n in ("ln1", "ln2"):
        t[n + "_g"], t[n + "_b"] = near(D, 1.0), near(D, 0.01)
    t["S_a"], t["attn_out_scale"] = near(f, 0.02), near(D, 1 / 255)
    t["w_2_bf16"] = (torch.randn((D, f), device="cuda", generator=g) * f ** -0.5).to(torch.bfloat16)
    return t, hero.layer_weights(t, 2e-4, 1 / 448 if mode & HB.M_FP8 else 1 / 255), \
        hero.layer_desc(HB.ARCH_PRE_LN, D, H, DH, f, 1e-5, HB.MASK_CAUSAL, mode)


@pytest.mark.parametrize("mode,B,S,f,planes", [
    (HB.MODE_M2, 1, 300, 16384, 8),                      # 16-bit FC2 of a chunk: 8 ranges of 300 x 1024 sums
    (HB.MODE_M2, 1, 200, 32768, 8),
    (HB.MODE_M3 | HB.M_FP8, 64, 1, 8192, 16),            # E4M3 FC2 of a decode step: 16 ranges
])
def test_split_scratch_of_fp32_sums_is_optional(mode, B, S, f, planes):
    hero = pkg.load()
    keep, W, desc = _layer(hero, mode, f, 5)
    T, full = B * S, hero.hero_layer_workspace_bytes(desc, B, S)
    least = full - planes * T * D * 4
    g = torch.Generator(device="cuda").manual_seed(6)
    h0 = torch.randn((T, D), device="cuda", generator=g).to(torch.bfloat16)

    def run(nbytes):
        h, ws = h0.clone(), torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        hero.hero_layer_fwd(desc, W, B, S, ws, h=h)
        return h.float()
    with_split, without, some = run(full), run(least), run(least + 4096)
    assert torch.equal(without, some)
    # the sums part by their fp32 order, a rounding to bf16 at most behind them
    assert float((with_split - without).norm() / with_split.norm()) <= 2.0 ** -8
    with pytest.raises(HB.HeroError) as e:
        run(least - 256)
    assert e.value.status == 5


def test_split_scratch_of_int8_is_needed():
    hero = pkg.load()
    keep, W, desc = _layer(hero, HB.MODE_M3, 8192, 7)
    h = torch.randn((64, D), device="cuda").to(torch.bfloat16)
    full = hero.hero_layer_workspace_bytes(desc, 64, 1)
    with pytest.raises(HB.HeroError) as e:
        hero.hero_layer_fwd(desc, W, 64, 1, torch.empty(full - 256, dtype=torch.uint8, device="cuda"), h=h)
    assert e.value.status == 5
    hero.hero_layer_fwd(desc, W, 64, 1, torch.empty(full, dtype=torch.uint8, device="cuda"), h=h)
    assert bool(torch.isfinite(h.float()).all())
