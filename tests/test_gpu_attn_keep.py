"""The one-pass attention of up to 512 keys (64 channels, 192 blocks of 128 queries or more) against the oracle: every number of
key tiles its body is unrolled for, tile edges +- 1, sequences shorter than the launch's tiles, and without keys."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB
from parity import assert_codes, fp8_attn_flip_bound, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("Sq,Skv,lens", [(65, 65, (65, 1)), (128, 128, (128, 63)), (40, 64, (64, 17)), (129, 129, (129, 64)), (192, 192, (192, 130)),
                                        (256, 256, (256, 193)), (257, 257, (257, 0)), (33, 320, (320, 65)), (384, 384, (384, 321)),
                                        (100, 449, (449, 385)), (512, 512, (512, 448))])
def test_against_oracle(Sq, Skv, lens, mask, fp8):
    H = 6
    against_oracle(256 // (H * ((Sq + 127) // 128)) + 1, H, Sq, Skv, lens, mask, fp8)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING])
@pytest.mark.parametrize("B,H,Sq,Skv,lens", [(48, 2, 160, 160, (160, 129)), (48, 2, 161, 161, (161, 100)), (21, 4, 320, 320, (320, 161)),
                                             (20, 4, 320, 320, (320, 161)), (128, 4, 300, 300, (300, 151)), (96, 4, 400, 400, (400, 257)),
                                             (127, 4, 300, 300, (300, 300)), (128, 4, 64, 400, (400, 65)), (129, 4, 64, 400, (400, 65)), (257, 4, 96, 260, (260, 250))])
def test_either_side_of_the_rules(B, H, Sq, Skv, lens, mask, fp8):
    against_oracle(B, H, Sq, Skv, lens, mask, fp8)                   # little filled blocks, crowded XCDs, E4M3 of many blocks or few queries


def against_oracle(B, H, Sq, Skv, lens, mask, fp8):
    hero, Dh = pkg.load(), 64
    g = torch.Generator(device="cuda").manual_seed(Sq * 3 + Skv)
    dt = torch.float8_e4m3fn if fp8 else torch.int8
    qkv = [(torch.randn((B, s, 3, H, Dh), device="cuda", generator=g) * (40 if fp8 else 30)).clamp(-127, 127).to(dt) for s in (Sq, Skv)]
    q, k, v = qkv[0][:, :, 0], qkv[1][:, :, 1], qkv[1][:, :, 2]     # rows of the packed projection
    if mask == HB.MASK_CAUSAL and Sq == Skv:
        lens = (Skv, Skv)                                           # prefill
    kv = torch.tensor([lens[b % 2] for b in range(B)], dtype=torch.int32, device="cuda")
    ps, qk = (1 / 448, 1.5 / (1600 * Dh ** 0.5)) if fp8 else (1 / 255, 3.0 / (900 * Dh ** 0.5))      # logits of a few units
    scale = torch.rand(H * Dh, device="cuda", generator=g) * 0.4 * ps + 0.8 * ps
    scale = scale * (4 if fp8 else 127 / 30 / 2.5)
    fn = hero.hero_fp8_attn if fp8 else hero.hero_int8_attn
    got = fn(q, k, v, qk, ps, scale, mask=mask, kv_len=kv).view(torch.int8).reshape(B, Sq, H * Dh)
    hp = fn(q, k, v, qk, ps, scale[:1].contiguous(), out_scale_is_scalar=True, mask=mask, kv_len=kv, out_dtype=torch.bfloat16).reshape(B, Sq, H * Dh)
    sel = [0, 1, B - 1]
    n = lambda t: np.ascontiguousarray(to_np(t.view(torch.int8)[sel]).view(np.uint8 if fp8 else np.int8))
    qn, kn, vn, kvn, sn = n(q), n(k), n(v), to_np(kv[sel]), to_np(scale)
    kw = dict(qk_scale=qk, p_scale=ps, mask=mask, kv_len=kvn)
    of = O.fp8_attn if fp8 else O.int8_attn
    ref = of(qn, kn, vn, out_col_scale=sn, **kw)
    refh = of(qn, kn, vn, out_col_scale=sn[:1].copy(), out_scale_is_scalar=True, out_dt=O.F32, **kw)
    g8 = to_np(got[sel]).reshape(ref.shape)
    if fp8:
        # possible flips + one step of the output grid + the error of the matrix cores' PV sums, which is roughly normal with 2.5e-4
        # of a typical sum (class 1e-3, i.e. four sigma: 6e-5 of the outputs lie beyond it, none at sixteen)
        D = fp8_attn_flip_bound(qn, kn, vn, qk, ps, sn, mask, kvn)
        x, o = O.e4m3_to_f32(g8.view(np.uint8)).astype(np.float64), O.e4m3_to_f32(ref).astype(np.float64)
        step = np.maximum(2.0 ** (np.floor(np.log2(np.maximum(np.abs(o), 2.0 ** -6))) - 3), 2.0 ** -9)
        excess = (np.abs(x - o) - 1.0001 * (D + step)) / np.sqrt(np.mean(o * o))
        assert excess.max() <= 4e-3 and np.mean(excess > 1e-3) <= 6e-5, (excess.max(), np.mean(excess > 1e-3))
    else:
        assert_codes(g8, ref)
        # a probability code that parts moves an output by one |v| <= 127 times the scale; the result is rounded to 16 bits
        d = np.abs(hp[sel].float().cpu().numpy().reshape(refh.shape) - refh)
        assert np.all(d <= 127.5 * sn[0] + 2.0 ** -8 * np.abs(refh)) and np.mean(d > 2.0 ** -8 * np.abs(refh) + 1e-5) <= 1e-3


@pytest.mark.parametrize("Skv", [200, 300, 513])
def test_a_nan_code_stays_with_its_key(Skv):
    """E4M3, one pass (200 and 300 keys) and two (513): a key that holds a NaN code gets the largest probability code and the row's other
    keys code 0, for the row has no sum to divide by.  Rows that do not see it are untouched."""
    hero, H, Dh, B = pkg.load(), 6, 64, 20
    g = torch.Generator(device="cuda").manual_seed(Skv)
    q, k, v = ((torch.randn((B, Skv, H, Dh), device="cuda", generator=g) * 40).to(torch.float8_e4m3fn) for _ in range(3))
    scale = torch.full((H * Dh,), 1 / 448 / 64, device="cuda")
    run = lambda key: hero.hero_fp8_attn(q, key, v, 1.5 / (1600 * 8), 1 / 448, scale).view(torch.int8).reshape(B, Skv, H, Dh)
    ref = run(k)
    bad = k.clone()
    bad.view(torch.int8)[3, 17, 2, 5] = 0x7F
    want = (448 * v[3, 17, 2].float() * scale[0]).to(torch.float8_e4m3fn).view(torch.int8)
    got = run(bad)
    assert bool((got[3, :, 2] == want).all())
    got[3, :, 2] = ref[3, :, 2]
    assert torch.equal(got, ref)
