"""16-bit attention, the kernel of many query blocks, against 64 bits: lengths around its tiles and waves, scales it folds into the exponent and others,
and probabilities below FP16's smallest normal number."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB

pytestmark = pytest.mark.gpu
DTYPES = [torch.bfloat16, torch.float16]


def _visible(B, Sq, Skv, mask, lens):
    rows, cols = torch.arange(Sq, device="cuda")[:, None], torch.arange(Skv, device="cuda")[None, :]
    n = lens.long()[:, None, None] if lens is not None else torch.full((B, 1, 1), Skv, device="cuda")
    if mask == HB.MASK_CAUSAL:
        return cols <= rows + (n - Sq)
    vis = (cols < n).expand(B, Sq, Skv)
    return vis & (rows < n) if mask == HB.MASK_PADDING and Sq == Skv else vis


def _check(q, k, v, scale, mask, lens):
    B, Sq, H, D = q.shape
    Skv, dt = k.shape[1], q.dtype
    y = pkg.load().hero_hp_attn(q, k, v, scale, mask, lens).double().reshape(B, Sq, H, D)
    q, k, v = (t.double().transpose(1, 2).contiguous() for t in (q, k, v))
    vis = _visible(B, Sq, Skv, mask, lens)[:, None]
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) * scale
    any_ = vis.any(3, keepdim=True)
    p = torch.softmax(s.masked_fill(~vis, -torch.inf).masked_fill(~any_, 0.0), 3) * any_
    ref, mag = torch.matmul(p, v).transpose(1, 2), torch.matmul(p, v.abs()).transpose(1, 2)
    peak = (torch.matmul((vis & any_).double().expand(B, H, Sq, Skv), v.abs())).transpose(1, 2)
    half = 2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -11           # half an ulp of 8 (11) significant bits, relative to the value at most
    # a probability and the result are rounded to 16 bits (FP16: of step 2^-24 below its smallest normal number, of the largest one); the
    # scores' fp32 sums are off by D 2^-24 of sum |q k| at most, and so are their exponentials, twice (the row sum)
    slack = 2 * (D + 8) * 2.0 ** -24 * abs(scale) * torch.matmul(q.abs(), k.abs().transpose(2, 3).contiguous()).amax(3).transpose(1, 2)[..., None]
    bound = (2 * half + slack + 1e-6) * mag + half * ref.abs() + (2.0 ** -25 * peak if dt == torch.float16 else 0) + 2.0 ** -25
    assert bool(((y - ref).abs() <= bound).all()), float(((y - ref).abs() / bound).max())


@pytest.mark.parametrize("dt", DTYPES)
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("mask", [HB.MASK_NONE, HB.MASK_PADDING, HB.MASK_CAUSAL])
@pytest.mark.parametrize("S", [33, 63, 64, 65, 127, 129, 200])
def test_lengths(S, mask, D, dt):
    g = torch.Generator(device="cuda").manual_seed(S + D)
    B, H = (40, 16) if S < 128 else (20, 16)
    q, k, v = (torch.randn((B, S, H, D), device="cuda", generator=g).to(dt) for _ in range(3))
    lens = None if mask == HB.MASK_NONE else torch.randint(0, S + 1, (B,), device="cuda", generator=g, dtype=torch.int32)
    if lens is not None:
        lens[:4] = torch.tensor([0, 1, S, S - 1], device="cuda")
    _check(q, k, v, D ** -0.5, mask, lens)


@pytest.mark.parametrize("dt", DTYPES)
@pytest.mark.parametrize("scale", [-0.125, 0.0, 1e-30, 0.7])
@pytest.mark.parametrize("mask", [HB.MASK_PADDING, HB.MASK_CAUSAL])
def test_scales(mask, scale, dt):
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((40, 100, 16, 64), device="cuda", generator=g).to(dt) for _ in range(3))
    _check(q, k, v, scale, mask, torch.randint(1, 101, (40,), device="cuda", generator=g, dtype=torch.int32))


@pytest.mark.parametrize("dt", DTYPES)
def test_small_probabilities(dt):
    """One key ahead of the others by 10: they hold 4.5e-5 each (a subnormal FP16 number) and 2 % together."""
    g = torch.Generator(device="cuda").manual_seed(9)
    q, k, v = torch.zeros((40, 128, 16, 64), device="cuda"), torch.zeros((40, 500, 16, 64), device="cuda"), torch.randn((40, 500, 16, 64), device="cuda", generator=g)
    q[..., 0], k[:, 77, :, 0], v[:, 77] = 1.0, 10.0, 0.0
    _check(q.to(dt), k.to(dt), (v + 1).to(dt), 1.0, HB.MASK_NONE, None)


@pytest.mark.parametrize("dt,unit,scale", [(torch.bfloat16, 1e19, 4.0), (torch.float16, 3e4, 4e29)])
@pytest.mark.parametrize("key", [5, 40, 99])
def test_a_score_beyond_fp32_is_not_silent(dt, unit, scale, key):
    """A sum that fp32 holds, times a scale that takes it beyond: the row has no maximum to subtract, and is NaN (as softmax of fp32 scores is), not zeros."""
    g = torch.Generator(device="cuda").manual_seed(9)
    q, k, v = torch.zeros((40, 100, 16, 64), device="cuda"), torch.zeros((40, 100, 16, 64), device="cuda"), torch.randn((40, 100, 16, 64), device="cuda", generator=g)
    q[3, 17, 2, 0], k[3, key, 2, 0] = unit, unit
    bad = torch.zeros(q.shape, device="cuda", dtype=torch.bool)
    bad[3, 17, 2] = True
    for n in (slice(0, 40), slice(3, 4)):                           # many query blocks, few
        y = pkg.load().hero_hp_attn(q[n].to(dt), k[n].to(dt), v[n].to(dt), scale, HB.MASK_NONE, None)
        assert torch.equal(torch.isnan(y).reshape(bad[n].shape), bad[n])
