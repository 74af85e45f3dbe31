"""8-bit attention: a query's keys are shared by two lanes (keys 0-3 of every eight with the one, 4-7 with the other), which have to agree on the row's
maximum.  One key far ahead of all others, at every position modulo eight, against the oracle; and the two kernels against each other where a
query's last tile shows keys to one of its two lanes only, or a few to the second."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB
from parity import to_np
from test_gpu_attn_split import test_split_against_block as against_split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("Sq,Skv", [(20, 150), (130, 600), (577, 577), (20, 1023), (90, 1024)])
def test_one_key_far_ahead(Dh, fp8, mask, Sq, Skv):
    """Query i asks for channel i % Dh, in which one key leads the others by 100 or 300 units of the softmax's exponent: that key's probability is 1, the others' 0,
    and the output is its V, code for code.  From 88.7 units (2^128) on a maximum that misses the key makes the row's sum infinite."""
    hero, B, H = pkg.load(), 2, 2
    if mask == HB.MASK_CAUSAL and Sq == Skv:
        Sq -= 500                                                   # every leading key has to be visible to every query
    g = torch.Generator(device="cuda").manual_seed(Sq + Skv)
    dt = torch.float8_e4m3fn if fp8 else torch.int8
    top, side, unit = (448.0, 96.0, 128.0) if fp8 else (127.0, 40.0, 127.0)
    lens = [Skv, Skv - 9] if mask != HB.MASK_CAUSAL else [Skv, Skv]
    nlead = min(lens) if mask != HB.MASK_CAUSAL else Skv - Sq + 1
    lead = [37 * c % nlead for c in range(Dh)]
    assert len(set(lead)) == Dh and {n % 8 for n in lead} == set(range(8))
    q = torch.zeros((B, Sq, H, Dh), device="cuda")
    q[:, torch.arange(Sq), :, torch.arange(Sq) % Dh] = unit
    k = (torch.randn((B, Skv, H, Dh), device="cuda", generator=g) * (side / 2)).clamp(-side, side)
    k[:, lead, :, torch.arange(Dh)] = top
    v = (torch.randn((B, Skv, H, Dh), device="cuda", generator=g) * 40).clamp(-127, 127)
    v = torch.where(v.abs() < 1, 1.0, v)                            # (no zeros: E4M3 has two)
    q, k, v = q.to(dt), k.to(dt), v.to(dt)
    kv = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ps = 1 / 448 if fp8 else 1 / 255
    scale = torch.full((H * Dh,), ps, device="cuda")
    fn, of = (hero.hero_fp8_attn, O.fp8_attn) if fp8 else (hero.hero_int8_attn, O.int8_attn)
    n = lambda t: np.ascontiguousarray(to_np(t.view(torch.int8)).view(np.uint8 if fp8 else np.int8))
    for gap in (100.0, 300.0):
        qk = gap / (unit * (top - side))
        ref = torch.from_numpy(of(n(q), n(k), n(v), qk_scale=qk, p_scale=ps, out_col_scale=to_np(scale), mask=mask, kv_len=to_np(kv)).view(np.int8)).cuda()
        for r in (1, 1024 // (B * H * ((Sq + 127) // 128)) + 1):      # few queries: the keys split over a block's waves; many blocks: two passes
            got = fn(*(t.repeat(r, 1, 1, 1) for t in (q, k, v)), qk, ps, scale, mask=mask, kv_len=kv.repeat(r)).view(torch.int8)
            assert torch.equal(got.view(r, -1), ref.reshape(1, -1).expand(r, -1)), (gap, r)


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("S", [516, 517, 521, 546, 548, 576])
def test_last_tile(Dh, fp8, mask, S):
    against_split(Dh, fp8, mask, S, S)
