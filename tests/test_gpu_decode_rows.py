"""The decode step's kernels at their edges: attention that appends this call's K / V row to the cache itself, and LN^quant
with a workgroup per row of 16-bit values."""
import pytest
import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB, prep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Dh", [(2, 64), (32, 64), (2, 128), (32, 128)])      # 10 and 160 blocks wide, 320 narrow below
@pytest.mark.parametrize("fmt", ["i8", "fp8"])
@pytest.mark.parametrize("B", [5, 10])
def test_append_in_attention(H, Dh, fmt, B):
    """A cache of 640 positions (one kernel) against the same sequences in a cache too long for that kernel (a copy of the
    row, then the general kernel): the same cache rows, outputs within the class of a 16-bit layer.  Lengths: the first
    token, a full cache, one past it (nothing is appended), the edges of the loops' rounds."""
    hero, d, f, mode = pkg.load(), H * Dh, 256, HB.MODE_M3 | (HB.M_FP8 if fmt == "fp8" else 0)
    g = torch.Generator(device="cuda").manual_seed(H + Dh)
    p = {k: torch.randn(s, device="cuda", generator=g) * d ** -0.5 for k, s in
         {"w_qkv": (d, 3 * d), "b_qkv": (3 * d,), "w_o": (d, d), "b_o": (d,), "w_1": (d, f), "b_1": (f,), "w_2": (f, d), "b_2": (d,)}.items()}
    for k in ("ln1", "ln2"):
        p[k + "_g"], p[k + "_b"] = torch.ones(d, device="cuda"), torch.zeros(d, device="cuda")
    x = torch.randn((2 * 64, d), device="cuda", generator=g).double()
    sc, _ = prep.calibrate(p, x, HB.ARCH_PRE_LN, H, Dh, 1e-5, HB.MASK_CAUSAL, 2, 64, hero=hero, fp8=fmt == "fp8")
    t, qk, ps = prep.prepare(p, sc, HB.ARCH_PRE_LN, d, Dh, HB.MODE_M3, hero=hero, fp8=fmt == "fp8")
    W, desc = hero.layer_weights(t, qk, ps), hero.layer_desc(HB.ARCH_PRE_LN, d, H, Dh, f, 1e-5, HB.MASK_CAUSAL, mode)
    short, long_ = 640, 16400
    kv = torch.tensor([1, 2, 513, short, 257, 256, 640, 31, 33, 64][:B], dtype=torch.int32, device="cuda")
    dt = torch.float8_e4m3fn if fmt == "fp8" else torch.int8
    full = [(torch.randn((B, H, long_, Dh), device="cuda", generator=g) * 30).clamp(-127, 127).to(dt) for _ in range(2)]
    h0 = torch.randn((B, d), device="cuda", generator=g).to(torch.bfloat16)
    outs = []
    for smax in (short, long_):
        ws = torch.empty(hero.hero_layer_workspace_bytes(desc, B, 1), dtype=torch.uint8, device="cuda")
        kc, vc = (c[:, :, :smax].contiguous() for c in full)
        h = h0.clone()
        hero.hero_layer_fwd(desc, W, B, 1, ws, h=h, kv_len=kv, k_cache=kc, v_cache=vc)
        outs.append((h.float(), kc[:, :, :short].contiguous().view(torch.int8), vc[:, :, :short].contiguous().view(torch.int8)))
    assert torch.equal(outs[0][1], outs[1][1]) and torch.equal(outs[0][2], outs[1][2])
    changed = (outs[0][1] != full[0][:, :, :short].contiguous().view(torch.int8)).any(3).any(1)           # [B, position]
    assert all(changed[b].nonzero().flatten().tolist() in ([int(kv[b]) - 1], []) for b in range(B))
    assert float((outs[0][0] - outs[1][0]).norm() / outs[1][0].norm()) <= 4e-3
    # nothing appended past the end or for an empty sequence; the empty one attends to nothing
    kc, vc, h = full[0][:, :, :short].contiguous(), full[1][:, :, :short].contiguous(), h0.clone()
    kv2 = kv.clone()
    kv2[0], kv2[1] = 0, short + 1
    hero.hero_layer_fwd(desc, W, B, 1, torch.empty(hero.hero_layer_workspace_bytes(desc, B, 1), dtype=torch.uint8, device="cuda"),
                        h=h, kv_len=kv2, k_cache=kc, v_cache=vc)
    assert torch.equal(kc[:2].view(torch.int8), full[0][:2, :, :short].contiguous().view(torch.int8))
    assert torch.equal(vc[:2].view(torch.int8), full[1][:2, :, :short].contiguous().view(torch.int8))
    assert bool(torch.isfinite(h.float()).all())


# cache lengths around the rounds and units of both block widths (a unit is 32 .. 128 keys, a round eight of them)
LENGTHS = [0, 1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 512, 513, 600, 1023, 1024, 1025, 1100]


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("fp8", [False, True])
def test_decode_attention_lengths(Dh, fp8):
    """One query per sequence against 64 bits, every length, from wide blocks (72 of them) and from narrow ones (the same again
    until there are more than 256)."""
    hero, B, H, cap = pkg.load(), len(LENGTHS), 3, 1100
    g = torch.Generator(device="cuda").manual_seed(Dh)
    dt = torch.float8_e4m3fn if fp8 else torch.int8
    draw = lambda S: (torch.randn((B, S, H, Dh), device="cuda", generator=g) * 30).clamp(-127, 127).to(dt)
    q, k, v = draw(1), draw(cap), draw(cap)
    kv = torch.tensor(LENGTHS, dtype=torch.int32, device="cuda")
    qk, ps = 0.08 / Dh ** 0.5 / 30, 1 / 448 if fp8 else 1 / 255
    one = torch.ones(1, device="cuda")
    fn = hero.hero_fp8_attn if fp8 else hero.hero_int8_attn
    call = lambda r: fn(*(t.repeat(r, 1, 1, 1) for t in (q, k, v)), qk, ps, one, out_scale_is_scalar=True, kv_len=kv.repeat(r),
                        out_dtype=torch.float16).reshape(r, B, H, Dh).double()
    a = (q.double() * k.double()).sum(3).transpose(1, 2) * qk                       # [B, H, cap]
    hidden = torch.arange(cap, device="cuda")[None, None, :] >= kv[:, None, None]
    p = torch.softmax(a.masked_fill(hidden, -1e300), 2) * (kv > 0)[:, None, None] / ps
    if fp8:
        step = 2.0 ** (torch.floor(torch.log2(p.clamp(min=2.0 ** -6))) - 3)
        p = ((p / step).round() * step).clamp(max=448)
    else:
        p = p.round()
    p = p.masked_fill(hidden, 0.0)
    ref = (p[..., None] * v.double().transpose(1, 2)).sum(2)                        # [B, H, Dh]
    # a probability code parts where it lies within fp32 rounding (6e-5 of a step) of a tie: about one in 2e4, by one step of at
    # most 1 (E4M3: 1 / 8 of its value), so a few of a row's keys move its outputs by some 1e2; then one rounding to fp16
    near = 3 * 127 * (p.amax(2, keepdim=True) / 8 if fp8 else torch.ones_like(p[..., :1]))
    for o in (call(1), call(4)):
        assert bool((o == o[:1]).all())
        d = (o[0] - ref).abs()
        assert bool((d <= near + ref.abs() * 2.0 ** -11 + 2.0 ** -14).all())
        close = d <= ref.abs() * 2.0 ** -10 + (1e-5 * p.sum(2, keepdim=True) * 448 if fp8 else 0.0) + 2.0 ** -14
        assert float((~close).any(2).float().mean()) <= 0.1                           # rows with any parted code
        assert bool((o[0, 0] == 0).all())


@pytest.mark.parametrize("D", [1040, 2048, 2064, 4096])
@pytest.mark.parametrize("M", [1, 3, 1537, 4000])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("fp8", [False, True])
def test_ln_quant_row_per_workgroup(D, M, dt, fp8):
    hero = pkg.load()
    g = torch.Generator(device="cuda").manual_seed(D + M)
    x = (torch.randn((M, D), device="cuda", generator=g) * 3 + 1).to(dt)
    x[0] = 2.0                                                     # no variance: the row is beta
    gamma, beta = 1 + 0.1 * torch.randn(D, device="cuda", generator=g), 0.1 * torch.randn(D, device="cuda", generator=g)
    odd = torch.empty(D + 1, device="cuda")
    odd[1:] = gamma
    ref = torch.nn.functional.layer_norm(x.double(), (D,), gamma.double(), beta.double(), 1e-5)
    s_ref = ref.abs().amax(1) / (448 if fp8 else 127)
    for gm in (gamma, odd[1:]):                                    # aligned for 128-bit loads, and not
        q, s, y = hero.hero_ln_quant(x, None, None, None, gm, beta, 1e-5, y_hp_dtype=dt, fp8=fp8)
        # fp32 statistics over D values: some 1e-6; the 16-bit copy is rounded once
        assert float(((s.double() - s_ref).abs() / s_ref).max()) <= 1e-5
        assert bool(((y.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 2e-5 * ref.abs().amax(1, keepdim=True)).all())
        z = ref / s_ref[:, None]
        if fp8:
            assert float(((q.double() - z).abs() / z.abs().clamp(min=2.0 ** -6)).max()) <= 2.0 ** -4 * 1.01   # half a step of 3 bits
        else:
            assert float((q.double() - z).abs().max()) <= 0.501
