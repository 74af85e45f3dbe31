"""Keys outside the mask where the scale of the scores vanishes, on every 8-bit attention kernel with a mask, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB
from parity import assert_codes, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("qk", [2.0 ** -23, 1e-9, 1e-38, 0.0])
@pytest.mark.parametrize("B,Sq,Skv,Dh", [(2, 513, 513, 64), (44, 97, 577, 64), (44, 97, 161, 128),
                                         (2, 65, 65, 64), (3, 33, 200, 128), (2, 17, 600, 64),
                                         # from here on: the one-pass kernel's sizes
                                         (43, 65, 65, 64), (22, 129, 129, 64), (15, 257, 257, 64), (11, 509, 509, 64), (43, 33, 320, 64)])
def test_hidden_keys_at_vanishing_scales(B, Sq, Skv, Dh, qk, mask, fp8):
    """With scores that tell no key from another a hidden key must be left out as such, not by the size of its score: padded keys and
    the future hold larger values than what a query sees.  S_p = 2^-8: no number of equal probabilities lies on a rounding tie."""
    hero, H = pkg.load(), 6
    g = torch.Generator(device="cuda").manual_seed(Sq + Skv)
    dt = torch.float8_e4m3fn if fp8 else torch.int8
    q, k = ((torch.randn((B, s, H, Dh), device="cuda", generator=g) * 30).clamp(-127, 127).to(dt) for s in (Sq, Skv))
    lens = [Skv if mask == HB.MASK_CAUSAL and Sq == Skv else n for n in (Skv - Skv // 3, Skv)]
    kv = torch.tensor([lens[b % 2] for b in range(B)], dtype=torch.int32, device="cuda")
    at = torch.arange(Skv, device="cuda")
    ramp = torch.where(at < kv[:, None], 5 + 60 * at // Skv, 120)
    v = (ramp[:, :, None, None] + torch.randint(-4, 5, (B, Skv, H, Dh), device="cuda", generator=g)).float().to(dt)
    scale = (torch.rand(H * Dh, device="cuda", generator=g) + 0.5) / 256
    fn, of = (hero.hero_fp8_attn, O.fp8_attn) if fp8 else (hero.hero_int8_attn, O.int8_attn)
    got = fn(q, k, v, qk, 2.0 ** -8, scale, mask=mask, kv_len=kv).view(torch.int8).reshape(B, Sq, H * Dh)
    sel = [0, 1, B - 1]
    n = lambda t: np.ascontiguousarray(to_np(t.view(torch.int8)[sel]).view(np.uint8 if fp8 else np.int8))
    ref = of(n(q), n(k), n(v), qk_scale=qk, p_scale=2.0 ** -8, out_col_scale=to_np(scale), mask=mask, kv_len=to_np(kv[sel]))
    g8 = to_np(got[sel]).reshape(ref.shape)
    if fp8:                                                          # one step of the output grid (the values are far from zero)
        x, o = O.e4m3_to_f32(g8.view(np.uint8)).astype(np.float64), O.e4m3_to_f32(ref).astype(np.float64)
        assert np.all(np.abs(x - o) <= 1.0001 * np.maximum(2.0 ** (np.floor(np.log2(np.maximum(np.abs(o), 2.0 ** -6))) - 3), 2.0 ** -9))
    else:
        assert_codes(g8, ref)
