"""What the performance of this library is measured on: W8A8 transformer layers as a serving program runs them (encoder
batches, prompts, prompt continuation, token generation), and the two operators a program calls on their own (the input
embedding and a stand-alone GeMM^quant).

Model shapes are the library's own: BERT-base (d 768), BERT-large (d 1024), the GPT-like decoder (d 4096), see
paper_2310_17723_amd/synth.py.  Values are drawn on the GPU from the distributions that module names: weights
N(0, w_std^2), activations N(0, 1) with a few outlier channels, LayerNorm gains 1 + N(0, 0.1^2); static scales come from
the library's own calibration, so the INT8 / E4M3 codes spread as they do behind it.
"""
from __future__ import annotations

import math

import torch

import paper_2310_17723_amd as pkg
from paper_2310_17723_amd import binding as HB
from paper_2310_17723_amd import prep, synth

MODELS = {"bert-base": synth.CONFIGS[0], "bert-large": synth.CONFIGS[2], "gpt": synth.CONFIGS[3]}
MODES = {"M0": HB.MODE_M0, "M1": HB.MODE_M1, "M2": HB.MODE_M2, "M3": HB.MODE_M3}
DTYPES = {"i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16}
ROOM = 128                       # positions of a KV cache beyond the sequences' present length (tokens still to come)
VOCAB, MAX_POS, TYPES = 30522, 512, 2


def _layer(name, model, B, S, mode="M3", hp="bf16", fmt="i8", lens="full", cache=0, layers=1):
    """B sequences of S new tokens through `layers` layers of the model.  lens: "full" = all sequences S long, "padded" =
    lengths in [S/2, S] under the padding mask.  cache: tokens per sequence already in the KV cache (0: no cache); with
    lens "ragged" each sequence holds between half of it and all of it."""
    c = {"kind": "layer", "model": model, "B": B, "S": S, "mode": mode, "hp": hp, "fmt": fmt, "lens": lens, "cache": cache,
         "layers": layers}
    return dict({"name": name} if name else {}, **c)


def _gemm(name, M, K, N, epi="dequant", out="f16"):
    return dict({"name": name} if name else {}, kind="gemm", M=M, K=K, N=N, epi=epi, out=out)


def _embed(name, model, B, S):
    return dict({"name": name} if name else {}, kind="embed", model=model, B=B, S=S)


def listed():
    return [
        # one short sentence through BERT-base: the smallest call, latency and launches decide
        _layer("bert-base-1x128", "bert-base", 1, 128),
        # a small batch of sentences of odd length with the attention side and FC2 in 16 bits (Table 1's M1)
        _layer("bert-base-7x93-m1", "bert-base", 7, 93, mode="M1", lens="padded"),
        # the headline: a full padded batch through a layer of BERT-large
        _layer("bert-large-32x512", "bert-large", 32, 512, lens="padded"),
        # the same batch in the mixed mode M1
        _layer("bert-large-32x512-m1", "bert-large", 32, 512, mode="M1", lens="padded"),
        # a middling batch of odd length with E4M3 as the 8-bit format
        _layer("bert-large-11x347-fp8", "bert-large", 11, 347, fmt="fp8", lens="padded"),
        # eight long prompts through a decoder layer: the largest call
        _layer("gpt-prefill-8x2048", "gpt", 8, 2048),
        # a chunk of two prompts continued on their caches, M2 with FP16 as the 16-bit type
        _layer("gpt-chunk-2x301-m2", "gpt", 2, 301, mode="M2", hp="f16", cache=900, lens="ragged"),
        # a full generation batch against 2048 cached tokens, two layers of the stack
        _layer("gpt-decode-64x1", "gpt", 64, 1, cache=2048, layers=2),
        # few users: three sequences generating
        _layer("gpt-decode-3x1", "gpt", 3, 1, cache=1500, lens="ragged", layers=2),
        # a generation batch with E4M3 codes and an E4M3 cache
        _layer("gpt-decode-24x1-fp8", "gpt", 24, 1, fmt="fp8", cache=1100, lens="ragged", layers=2),
        # a linear layer on its own: the long contraction of an FFN, 16-bit output, a row count no tile divides
        _gemm("gemm-2000x4096x1024", 2000, 4096, 1024),
        # the input stage of an encoder: token, position and sentence-type rows -> LN^quant
        _embed("embed-32x512", "bert-large", 32, 512),
    ]


def draw(rng):
    def logint(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(("bert", "bert", "bert", "prefill", "chunk", "decode", "decode", "gemm", "embed"))
    fmt = "fp8" if rng.random() < 0.2 else "i8"
    hp = rng.choice(("bf16", "bf16", "f16")) if fmt == "i8" else "bf16"
    mode = "M3" if fmt == "fp8" else rng.choice(("M0", "M1", "M2", "M3", "M3", "M3"))
    if kind == "bert":
        model = rng.choice(("bert-base", "bert-large"))
        S = logint(16, 512)
        B = logint(1, min(32, 16384 // S))
        return _layer(None, model, B, S, mode=mode, hp=hp, fmt=fmt, lens=rng.choice(("full", "padded", "padded")))
    if kind == "prefill":
        S = logint(32, 2048)
        B = logint(1, max(1, min(8, 8192 // S)))
        return _layer(None, "gpt", B, S, mode=mode, hp=hp, fmt=fmt)
    if kind in ("chunk", "decode"):          # the cache holds 8-bit codes: the attention module is 8-bit
        mode = rng.choice(("M2", "M3", "M3", "M3")) if fmt == "i8" else "M3"
        B, S = (logint(1, 8), logint(2, 512)) if kind == "chunk" else (logint(1, 64), 1)
        return _layer(None, "gpt", B, S, mode=mode, hp=hp, fmt=fmt, cache=logint(32, 2048), lens=rng.choice(("full", "ragged", "ragged")))
    if kind == "gemm":
        K, N = rng.choice(synth.GEMM_KN)
        epi, out = rng.choice((("dequant", "f16"), ("dequant", "bf16"), ("requant", "i8"), ("gelu", "i8")))
        return _gemm(None, logint(16, 8192), K, N, epi, out)
    S = logint(16, 512)
    return _embed(None, rng.choice(("bert-base", "bert-large")), logint(1, min(32, 16384 // S)), S)


# ---------------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(shape, device="cuda", generator=g)


def _params(g, sh):
    """fp32 parameters of one layer, the distributions of synth.layer_params."""
    d, f, s = sh.d, sh.f, sh.w_std
    p = {"w_qkv": (d, 3 * d), "b_qkv": (3 * d,), "w_o": (d, d), "b_o": (d,), "w_1": (d, f), "b_1": (f,), "w_2": (f, d), "b_2": (d,)}
    p = {k: _randn(g, *v) * s for k, v in p.items()}
    for k in ("ln1", "ln2"):
        p[k + "_g"], p[k + "_b"] = 1 + 0.1 * _randn(g, d), 0.02 * _randn(g, d)
    return p


def _hidden(g, sh, tokens, gain):
    return _randn(g, tokens, sh.d) * gain


def _prepare_layer(case, seed):
    hero, sh, g = pkg.load(), MODELS[case["model"]], _gen(seed)
    B, S, d, fp8 = case["B"], case["S"], sh.d, case["fmt"] == "fp8"
    T, post, cache = B * S, sh.arch == synth.POST_LN, case["cache"]
    mode = MODES[case["mode"]] | (HB.M_F16 if case["hp"] == "f16" else 0)
    hp = DTYPES[case["hp"]]
    gain = torch.ones(d, device="cuda")
    gain[torch.randperm(d, device="cuda", generator=g)[: round(sh.outlier_frac * d)]] = sh.outlier_mult
    emb_g, emb_b = 1 + 0.1 * _randn(g, d), 0.02 * _randn(g, d)
    mask = HB.MASK_CAUSAL if not post else (HB.MASK_PADDING if case["lens"] == "padded" else HB.MASK_NONE)

    # calibration on a small batch of its own, pushed through the unquantized layers
    Bc, Sc = 2, 64
    xc = _hidden(g, sh, Bc * Sc, gain).double()
    if post:
        xc = torch.nn.functional.layer_norm(xc, (d,), emb_g.double(), emb_b.double(), sh.eps)
    weights, keep, scales = [], [], []
    for _ in range(case["layers"]):
        p = _params(g, sh)
        sc, xc = prep.calibrate(p, xc, sh.arch, sh.H, sh.Dh, sh.eps, HB.MASK_NONE if post else HB.MASK_CAUSAL, Bc, Sc, hero=hero, fp8=fp8)
        t, qk, ps = prep.prepare(p, sc, sh.arch, d, sh.Dh, mode, hero=hero, fp8=fp8)
        keep.append(t)
        scales.append((qk, ps))
        weights.append(hero.layer_weights(t, qk, ps))
        del p

    desc = hero.layer_desc(sh.arch, d, sh.H, sh.Dh, sh.f, sh.eps, mask, mode | (HB.M_FP8 if fp8 else 0))
    st = {"kind": "layer", "hero": hero, "desc": desc, "weights": weights, "keep": keep, "scales": scales, "B": B, "S": S, "post": post,
          "next": [keep[(l + 1) % len(keep)].get("w_qkv") for l in range(len(keep))],
          "ws": torch.empty(hero.hero_layer_workspace_bytes(desc, B, S), dtype=torch.uint8, device="cuda")}
    h0 = _hidden(g, sh, T, gain)
    st["kv_len"] = st["caches"] = None
    if case["lens"] == "padded":
        st["kv_len"] = torch.randint((S + 1) // 2, S + 1, (B,), dtype=torch.int32, device="cuda", generator=g)
    if post:
        q, s, x = hero.hero_ln_quant(h0.to(hp), None, None, None, emb_g, emb_b, sh.eps, y_hp_dtype=hp, fp8=fp8)
        st["x"] = (q, s, x)
        st["bufs"] = [(torch.empty_like(q), torch.empty_like(s), None if mode & HB.M_QKV else torch.empty_like(x)) for _ in range(2)]
    else:
        st["h0"] = h0.to(hp)
        st["h"] = torch.empty_like(st["h0"])
    if cache:
        smax = cache + S + ROOM
        held = torch.randint((cache + 1) // 2, cache + 1, (B,), device="cuda", generator=g) if case["lens"] == "ragged" else \
            torch.full((B,), cache, device="cuda")
        st["kv_len"] = (held + S).to(torch.int32)
        st["caches"] = []
        for _ in range(case["layers"]):      # codes of a calibrated, roughly normal tensor: the largest of many values is 127 (448)
            kv = []
            for _ in range(2):
                c = torch.empty((B, sh.H, smax, sh.Dh), dtype=torch.float8_e4m3fn if fp8 else torch.int8, device="cuda")
                for b in range(B):
                    r = _randn(g, sh.H, smax, sh.Dh)
                    c[b] = (r * 100).clamp(-448, 448).to(c.dtype) if fp8 else (r * 30).round().clamp(-127, 127).to(c.dtype)
                kv.append(c)
            st["caches"].append(kv)
    return st


def _prepare_gemm(case, seed):
    g, M, K, N = _gen(seed), case["M"], case["K"], case["N"]
    codes = lambda n: (_randn(g, n, K) * 35).round().clamp(-127, 127).to(torch.int8)
    unif = lambda n: torch.rand(n, device="cuda", generator=g) * 1.5 + 0.5
    st = {"kind": "gemm", "hero": pkg.load(), "A": codes(M), "Bt": codes(N), "rs": unif(M) / 35,
          "cs": unif(N) / (35 * math.sqrt(K)), "bias": 0.02 * _randn(g, N), "out_scale": None,
          "epi": {"dequant": HB.EPI_DEQUANT, "requant": HB.EPI_REQUANT, "gelu": HB.EPI_GELU_REQUANT}[case["epi"]],
          "C": torch.empty((M, N), dtype=DTYPES[case["out"]], device="cuda")}
    if case["epi"] == "requant":             # the folded scale of the consumer: outputs spread over the codes
        st["cs"] = st["cs"] * 30
        st["bias"] = st["bias"] * 30
    if case["epi"] == "gelu":
        st["out_scale"] = unif(N) / 30
    return st


def _prepare_embed(case, seed):
    g, sh = _gen(seed), MODELS[case["model"]]
    B, S, d = case["B"], case["S"], sh.d
    tok = _randn(g, VOCAB, d) * 0.02
    scale = tok.abs().amax(1) / 127
    u = torch.rand(B * S, device="cuda", generator=g, dtype=torch.float64)
    ids = 10 * (((VOCAB + 10) / 10) ** u - 1)                  # word frequencies fall as 1 / (rank + 10)
    st = {"kind": "embed", "hero": pkg.load(), "tok": (tok / scale[:, None]).round().to(torch.int8), "tok_scale": scale,
          "pos": (0.02 * _randn(g, MAX_POS, d)).to(torch.bfloat16), "type": (0.02 * _randn(g, TYPES, d)).to(torch.bfloat16),
          "g": 1 + 0.1 * _randn(g, d), "b": 0.02 * _randn(g, d), "eps": sh.eps,
          "ids": ids.clamp(0, VOCAB - 1).to(torch.int32),
          "pos_ids": torch.arange(S, device="cuda", dtype=torch.int32).repeat(B),
          "y": (torch.empty((B * S, d), dtype=torch.int8, device="cuda"), torch.empty(B * S, device="cuda"))}
    split = torch.randint(S // 4, S, (B, 1), device="cuda", generator=g)
    st["type_ids"] = (torch.arange(S, device="cuda")[None, :] >= split).to(torch.int32).reshape(-1)
    return st


def prepare(case, seed):
    st = {"layer": _prepare_layer, "gemm": _prepare_gemm, "embed": _prepare_embed}[case["kind"]](case, seed)
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------------------------------------------- one pass
def run(st):
    hero = st["hero"]
    if st["kind"] == "gemm":
        return hero.hero_int8_gemm(st["A"], st["Bt"], st["rs"], st["cs"], st["bias"], epi=st["epi"], out_col_scale=st["out_scale"], C_out=st["C"])
    if st["kind"] == "embed":
        return hero.hero_embed_ln_quant(st["ids"], st["pos_ids"], st["type_ids"], st["tok"], st["tok_scale"], st["pos"], st["type"],
                                        st["g"], st["b"], st["eps"], y_q=st["y"][0], y_scale=st["y"][1])
    B, S, L = st["B"], st["S"], len(st["weights"])
    if st["post"]:
        xq, xs, xh = st["x"]
        for l in range(L):
            oq, os_, oh = st["bufs"][l & 1]
            hero.hero_layer_fwd(st["desc"], st["weights"][l], B, S, st["ws"], x_q=xq, x_scale=xs, x_hp=xh, out_q=oq, out_scale=os_,
                                out_hp=oh, kv_len=st["kv_len"], next_read=st["next"][l])
            xq, xs, xh = oq, os_, oh
        return [t for t in (xq, xs, xh) if t is not None]
    st["h"].copy_(st["h0"])
    for l in range(L):
        kc, vc = st["caches"][l] if st["caches"] else (None, None)
        hero.hero_layer_fwd(st["desc"], st["weights"][l], B, S, st["ws"], h=st["h"], kv_len=st["kv_len"], k_cache=kc, v_cache=vc,
                            next_read=st["next"][l])
    return [st["h"]] + [c for kv in st["caches"] or [] for c in kv]


# ---------------------------------------------------------------------------------------------------- the same in 64 bits
def _f8(x):
    """E4M3 values nearest to x, saturating: the codes lie on the grid 2^-9 * integers, 3 bits behind the leading one."""
    e = torch.floor(torch.log2(x.abs().clamp(min=2.0 ** -6)))
    u = torch.exp2(e - 3)
    return ((x / u).round() * u).clamp(-448, 448)


def _code(x, fp8):
    return _f8(x) if fp8 else x.round().clamp(-127, 127)


def _ln_quant64(x, g, b, eps, fp8):
    """LN^quant in 64 bits: codes, token-wise scales and the values themselves."""
    y = torch.nn.functional.layer_norm(x, x.shape[-1:], g.double(), b.double(), eps)
    s = y.abs().amax(1) / (448.0 if fp8 else 127.0)
    s = torch.where(s == 0, torch.ones_like(s), s)
    return _code(y / s[:, None], fp8), s, y


def _attn64(q, k, v, qk, ps, visible, fp8):
    """Attention of one sequence, [H, S, Dh] against [H, Skv, Dh]; ps: the step of the 8-bit probabilities (None: 16-bit
    attention).  visible: [S, Skv].  Rows that see nothing are zero."""
    out = torch.empty_like(q)
    any_ = visible.any(1)
    for h in range(q.shape[0]):
        a = (q[h] @ k[h].t()) * qk
        a = a.masked_fill(~visible, -torch.inf).masked_fill(~any_[:, None], 0.0)
        p = torch.softmax(a, 1) * any_[:, None]
        if ps is not None:
            p = _f8(p / ps) if fp8 else (p / ps).round().clamp(0, 255)
        out[h] = p @ v[h]
    return out


def _layer64(case, st, l, x, x_scale):
    """One layer in 64 bits: x are the input's codes with x_scale, or (pre-LN; a 16-bit QKV) its values.  The 8-bit codes and
    the 16-bit storage between two modules are the method's own and stay; everything between them is 64 bits."""
    sh, m, t = MODELS[case["model"]], MODES[case["mode"]], st["keep"][l]
    (qk, ps), fp8, post = st["scales"][l], case["fmt"] == "fp8", st["post"]
    B, S, d, H, Dh = st["B"], st["S"], sh.d, sh.H, sh.Dh
    hp = lambda v: v.to(DTYPES[case["hp"]]).double()
    D = lambda name: t[name].double()
    on = lambda bit: bool(m & bit)
    ln = lambda v, n: _ln_quant64(v, t[n + "_g"], t[n + "_b"], sh.eps, fp8)

    def linear(a, a_scale, w, w_hp, b, i8):
        y = a @ (D(w) if i8 else D(w_hp)).t()
        if i8:
            y = y * D(w + "_s")
            y = y if a_scale is None else y * a_scale[:, None]
        return y + D(b)

    h = x
    if post:
        xin, xs = x, x_scale
    else:
        c, s_, y = ln(h, "ln1")
        xin, xs = (c, s_) if on(HB.M_QKV) else (hp(y), None)
    qkv = linear(xin, xs, "w_qkv", "w_qkv_hp", "b_qkv", on(HB.M_QKV))
    qkv = _code(qkv, fp8) if on(HB.M_ATTN) else hp(qkv)
    q, k, v = (p.reshape(B, S, H, Dh).transpose(1, 2) for p in qkv.split(d, 1))
    caches = st["caches"][l] if st["caches"] else None
    rows = torch.arange(S, device="cuda")[:, None]
    attn = torch.empty((B, S, H, Dh), dtype=torch.float64, device="cuda")
    for b in range(B):
        n = int(st["kv_len"][b]) if st["kv_len"] is not None else S
        kb, vb = k[b], v[b]
        if caches:
            for c, new in zip(caches, (kb, vb)):
                c[b, :, n - S:n] = new.float().to(c.dtype)
            kb, vb = (c[b, :, :n].double() for c in caches)
        cols = torch.arange(kb.shape[1], device="cuda")[None, :]
        visible = (cols < n) & (rows < n) if post else cols <= rows + (n - S)
        attn[b] = _attn64(q[b], kb, vb, qk, ps if on(HB.M_ATTN) else None, visible, fp8).transpose(0, 1)
    attn = attn.reshape(B * S, d)
    if on(HB.M_ATTN):
        attn = attn * D("attn_out_scale")
    attn = _code(attn, fp8) if on(HB.M_ATTN_OUT) else hp(attn)
    o = linear(attn, None, "w_o", "w_o_bf16", "b_o", on(HB.M_ATTN_OUT))
    if post:
        o = _code(o, fp8) * D("S_o") if on(HB.M_ATTN_OUT) else hp(o)
        c, s_, y = ln((x * x_scale[:, None] if x_scale is not None else x) + o, "ln1")
    else:
        h = hp(h + o)
        c, s_, y = ln(h, "ln2")
    mid, ms = (c, s_) if on(HB.M_FC1) else (hp(y), None)
    a = torch.nn.functional.gelu(linear(mid, ms, "w_1", "w_1_hp", "b_1", on(HB.M_FC1)))
    a = _code(a / D("S_a"), fp8) if on(HB.M_FC2) else hp(a)
    x2 = linear(a, None, "w_2", "w_2_bf16", "b_2", on(HB.M_FC2))
    if not post:
        return hp(h + x2), None, None
    x2 = _code(x2, fp8) * D("S_x2") if on(HB.M_FC2) else hp(x2)
    return ln((mid * ms[:, None] if ms is not None else mid) + x2, "ln2")


def exact(case, seed):
    st = prepare(case, seed)
    if st["kind"] == "gemm":
        y = (st["A"].double() @ st["Bt"].double().t()) * st["rs"].double()[:, None] * st["cs"].double() + st["bias"].double()
        if case["epi"] == "gelu":
            y = torch.nn.functional.gelu(y) / st["out_scale"].double()
        return _code(y, False) if case["out"] == "i8" else y
    if st["kind"] == "embed":
        x = st["tok"][st["ids"].long()].double() * st["tok_scale"][st["ids"].long()].double()[:, None]
        x = x + st["pos"][st["pos_ids"].long()].double() + st["type"][st["type_ids"].long()].double()
        return _ln_quant64(x, st["g"], st["b"], st["eps"], False)[:2]
    if not st["post"]:
        h = st["h0"].double()
        for l in range(case["layers"]):
            h = _layer64(case, st, l, h, None)[0]
        return [h] + [c for kv in st["caches"] or [] for c in kv]
    q, s, y = st["x"]
    i8 = bool(MODES[case["mode"]] & HB.M_QKV)
    x, xs = (q.double(), s.double()) if i8 else (y.double(), None)
    for l in range(case["layers"]):
        q, s, y = _layer64(case, st, l, x, xs)
        x, xs = (q, s) if i8 else (y, None)
    return [q, s] if i8 else [q, s, y]


# ---------------------------------------------------------------------------------------------------- what a pass needs
def work(case):
    if case["kind"] == "gemm":
        M, K, N = case["M"], case["K"], case["N"]
        es = 1 if case["out"] == "i8" else 2
        return {"bytes": M * K + N * K + es * M * N + 4 * (M + (3 if case["epi"] == "gelu" else 2) * N), "flops": 2.0 * M * N * K}
    sh = MODELS[case["model"]]
    d, f, T = sh.d, sh.f, case["B"] * case["S"]
    if case["kind"] == "embed":
        return {"bytes": T * (2 * d + 20) + (case["S"] + TYPES) * 2 * d + 8 * d, "flops": 10.0 * T * d}
    m = MODES[case["mode"]]
    e = lambda bit: 1 if m & bit else 2
    weights = 3 * d * d * e(HB.M_QKV) + d * d * e(HB.M_ATTN_OUT) + d * f * (e(HB.M_FC1) + e(HB.M_FC2)) + 4 * (2 * (3 * d + d + f + d) + 4 * d)
    share = 0.75 if case["lens"] in ("padded", "ragged") else 1.0             # mean of lengths uniform in [1/2, 1]
    S, post = case["S"], sh.arch == synth.POST_LN
    held = case["cache"] * share
    seen = S * share if post else held + (S + 1) / 2                          # keys a query sees, on average
    pairs = case["B"] * S * (share if post else 1.0) * seen
    flops = 2.0 * T * (4 * d * d + 2 * d * f) + 4.0 * pairs * d
    cache_bytes = case["B"] * 2 * d * (held + 2 * S) if case["cache"] else 0  # the history read, this call's rows written
    io = T * (2 * d + 8) if post else 4 * T * d
    return {"bytes": case["layers"] * (weights + cache_bytes) + io, "flops": case["layers"] * flops}


def tolerance(case):
    """About four times what a pass differs from itself when every fp32 scale, gain and bias is moved by one unit in the
    last place (its sums rounded another way), over many shapes of the ranges drawn above.  A layer is discontinuous at
    code level: one flipped LN^quant or GELU^quant code moves a row of the following contraction."""
    if case["kind"] == "gemm":               # integer contraction, epilogue in one pinned fp32 order; GELU is fp32
        return {"rel": 0.0, "differ": 4e-4} if case["epi"] == "gelu" else "exact"
    if case["kind"] == "embed":              # measured: scales 1.1e-7, codes 6e-6
        return {"rel": 5e-7, "max": 2e-6, "differ": 4e-5}
    if case["fmt"] == "fp8":                 # measured: rel 3.2e-3, max 0.25 (a probability code on its neighbour's value)
        return {"rel": 1.3e-2, "max": 0.99, "differ": 1e-3}
    if case["mode"] in ("M0", "M1"):         # 16-bit attention against the same in 64 bits: codes 5e-3, attention output 2e-3
        return {"rel": 4e-3, "max": 0.05, "differ": 1e-2}
    if case["model"] == "gpt":               # measured: 16-bit stream rel 9e-4, max 1.3e-2; appended cache codes 9e-5
        return {"rel": 4e-3, "max": 0.05, "differ": 4e-4}
    return {"rel": 3e-4, "max": 0.03, "differ": 2e-3}      # measured: scales rel 6e-5, max 5.6e-3; codes 4.7e-4
