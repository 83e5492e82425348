"""The work that users of the encoder have it do, as cases to time and compare.

Every case goes through the public entry points (TextEncoder, build_positions,
VisionEncoder) eagerly, the way a program calls them. Shapes are the model
shapes of this repository: the Qwen3-VL-2B-class decoder (hidden 2048, 16 q / 8
kv heads of 128, FFN 6144, 28 layers), its tiny fp32 sibling, and the ViT tower
(width 1024, 16 heads of 64, MLP 4096). Weights and inputs are synthetic draws
of the distributions of synth/: linear weights and embeddings N(0, 0.02), norm
gains 1 + U(-0.5, 0.5), pixels N(0, 1); residual streams that enter a single
layer N(0, 1), the size they have after the first layer of such a stack.

listed() is the fixed set, draw() gives further cases of the same ranges,
prepare() what a program holds before the call, run() one call, work() what it
cannot do without, exact() the same result in float64 plain torch, tolerance()
how far two correct implementations at this precision may be apart.
"""
from __future__ import annotations

import math

import torch

from paper_2606_05981_amd import binding as B
from paper_2606_05981_amd.encoder import TextEncoder, VisionEncoder, build_positions

FULL = dict(hidden=2048, hq=16, hkv=8, hd=128, ffn=6144, sections=(24, 20, 20))
TINY = dict(hidden=256, hq=4, hkv=2, hd=64, ffn=768, sections=(12, 10, 10))
VIT = dict(hidden=1024, heads=16, hd=64, ffn=4096, patch=16, merge=2, channels=3, out=2048)
EPS, THETA, VIT_THETA = 1e-6, 5e6, 1e4


def _text(name, kind, lens, layers=1, dtype="bf16", weights="dtype", qk_norm=1, layout=0, prefix=0):
    """A text-encoder case. kind: "layer" (encode_layers of one layer on an fp32 residual
    stream), "encode" (build_positions + encode of the whole stack) or "prefixed"
    (encode_prefixed, `prefix` shared tokens). lens: "96x16" or "33,96,1"."""
    c = {"kind": kind, "lens": lens, "layers": layers, "dtype": dtype, "weights": weights, "qk_norm": qk_norm,
         "layout": layout, "prefix": prefix}
    return dict(c, name=name) if name else c


def _vision(name, images, height, width, depth=2):
    c = {"kind": "vision", "images": images, "height": height, "width": width, "depth": depth}
    return dict(c, name=name) if name else c


# 32 sequences of 102 .. 319 tokens (the mixed batch of synth.workloads)
MIXED = ("126,124,275,208,228,231,256,102,205,129,186,304,219,111,218,125,"
         "265,309,316,235,291,179,128,211,195,245,319,157,288,127,174,273")


def listed():
    return [
        # The smallest call: the tiny fp32 decoder (2 layers) on one 32-token sequence, all
        # launches and latency.
        _text("tiny_f32_1x32", "encode", "32", layers=2, dtype="f32"),
        # One decoder layer, one 256x256 frame with its instruction: what a stream that encodes
        # frame by frame pays 28 times; weights stream from memory.
        _text("layer_1x96", "layer", "96"),
        # The same with e4m3 weights, the option for this single-frame stage.
        _text("layer_1x96_e4m3", "layer", "96", weights="e4m3"),
        # A few requests of unequal length, packed: odd sizes, sequences that start inside tiles.
        _text("layer_5_ragged", "layer", "33,96,1,130,77"),
        # One layer of the batched dispatch, 16 frames of 96 tokens.
        _text("layer_16x96", "layer", "96x16"),
        # The same with e4m3 weights.
        _text("layer_16x96_e4m3", "layer", "96x16", weights="e4m3"),
        # One layer of a ragged batch of 32 sequences of mixed image sizes.
        _text("layer_mixed32", "layer", MIXED),
        # The largest layer: 32 frames of a 512x512 source (320 tokens each).
        _text("layer_32x320", "layer", "320x32"),
        # 16 frames behind one shared 80-token system prompt, encoded once (2 layers).
        _text("prefixed_16x96", "prefixed", "96x16", layers=2, prefix=80),
        # The vision tower on the 16 source frames of a batch: patch extraction, 2 of its 24
        # blocks, merger.
        _vision("vision_16x256", 16, 256, 256),
        # The whole encoder, 28 layers, one frame: positions to final norm.
        _text("stack28_1x96", "encode", "96", layers=28),
        # The whole encoder on the 16-frame batch, the framework's headline workload.
        _text("stack28_16x96", "encode", "96x16", layers=28),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _lens(rng, most):
    """Sequence lengths of a batch of at most `most` tokens: one, a few or many sequences, of 1
    to 320 tokens each, equal or not."""
    total = _log_int(rng, 8, most)
    n = max(1, min(_log_int(rng, 1, 32), total))
    top = min(320, max(1, 2 * total // n))
    if rng.random() < 0.3:
        return "%dx%d" % (max(1, min(320, total // n)), n)
    lens = []
    for _ in range(n):
        L = rng.randint(max(1, top // 4), top)
        if sum(lens) + L > most:
            break
        lens.append(L)
    return ",".join(str(x) for x in lens or [min(most, 77)])


def draw(rng):
    r = rng.random()
    if r < 0.08:
        return _text("", "encode", _lens(rng, 512), layers=2, dtype="f32", qk_norm=rng.randint(0, 1),
                     layout=rng.randint(0, 1))
    if r < 0.70:
        return _text("", "layer", _lens(rng, 10240), weights="e4m3" if rng.random() < 0.25 else "dtype",
                     qk_norm=0 if rng.random() < 0.1 else 1, layout=1 if rng.random() < 0.2 else 0)
    if r < 0.78:
        return _text("", "prefixed", _lens(rng, 3072), layers=rng.randint(1, 3), prefix=_log_int(rng, 1, 160))
    if r < 0.93:
        h, w = 32 * rng.randint(2, 16), 32 * rng.randint(2, 16)
        n = max(1, min(_log_int(rng, 1, 16), 4096 * 256 // (h * w)))
        return _vision("", n, h, w, depth=rng.randint(1, 3))
    return _text("", "encode", _lens(rng, 1536), layers=rng.randint(3, 28))


# ------------------------------------------------------------------ inputs
def _seq_lens(text):
    out = []
    for part in text.split(","):
        n, _, times = part.partition("x")
        out += [int(n)] * int(times or 1)
    return out


def _layout(length):
    """A sequence of `length` tokens as an image grid and its instruction (text only when short)."""
    text = 32 if length < 256 else 64
    side = int(math.isqrt(max(0, length - text)))
    if side < 2:
        return (0, 0, 0, 0, length)
    grid_w = min(16, (length - text) // side)
    return (0, 1, side, grid_w, length - side * grid_w)


def _positions(layouts, start=0):
    """(t, h, w) positions as int64 [3, T] on the host; text counts on after the largest used."""
    rows = []
    for _, _, gh, gw, n in layouts:
        rows += [(start, start + k // gw, start + k % gw) for k in range(gh * gw)]
        nxt = start + (max(gh, gw) if gh * gw else 0)
        rows += [(nxt + i,) * 3 for i in range(n)]
    return torch.tensor(rows, dtype=torch.int64).reshape(-1, 3).t().contiguous()


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt * 7919 + 17) % (1 << 62))
    return g


def _normal(g, shape, dt, std=0.02):
    return (torch.randn(shape, generator=g, device="cuda") * std).to(dt)


def _gain(g, n, dt):
    return (torch.rand(n, generator=g, device="cuda") + 0.5).to(dt)


def _dims(case):
    return TINY if case["dtype"] == "f32" else FULL


def _dt(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _layer(case, seed, l):
    m, g, dt = _dims(case), _gen(seed, 100 + l), _dt(case)
    D, q, kv, F, d = m["hidden"], m["hq"] * m["hd"], m["hkv"] * m["hd"], m["ffn"], m["hd"]
    return {"attn_norm": _gain(g, D, dt), "w_q": _normal(g, (q, D), dt), "w_k": _normal(g, (kv, D), dt),
            "w_v": _normal(g, (kv, D), dt), "q_norm": _gain(g, d, dt), "k_norm": _gain(g, d, dt),
            "w_o": _normal(g, (D, q), dt), "mlp_norm": _gain(g, D, dt), "w_gate": _normal(g, (F, D), dt),
            "w_up": _normal(g, (F, D), dt), "w_down": _normal(g, (D, F), dt)}


def _inputs(case, seed):
    """Everything drawn from the seed but the layers' weights."""
    if case["kind"] == "vision":
        g = _gen(seed, 1)
        D, mm, kp = VIT["hidden"], VIT["merge"] ** 2, VIT["channels"] * VIT["patch"] ** 2
        bf = torch.bfloat16
        outer = {"patch_w": _normal(g, (D, kp), bf), "patch_b": _normal(g, (D,), bf), "merge_ln_g": _gain(g, D, bf),
                 "merge_ln_b": _normal(g, (D,), bf, 0.1), "merge_w1": _normal(g, (mm * D, mm * D), bf),
                 "merge_b1": _normal(g, (mm * D,), bf), "merge_w2": _normal(g, (VIT["out"], mm * D), bf),
                 "merge_b2": _normal(g, (VIT["out"],), bf)}
        px = _normal(_gen(seed, 2), (case["images"], VIT["channels"], case["height"], case["width"]), bf, 1.0)
        return {"outer": outer, "pixels": px}
    lens, dt, D = _seq_lens(case["lens"]), _dt(case), _dims(case)["hidden"]
    T = sum(lens)
    x = {"final": _gain(_gen(seed, 3), D, dt)}
    if case["kind"] == "layer":
        x["h"] = _normal(_gen(seed, 4), (T, D), torch.float32, 1.0)
    else:
        x["embeds"] = _normal(_gen(seed, 4), (T, D), dt)
    if case["kind"] == "prefixed":
        x["prefix"] = _normal(_gen(seed, 5), (case["prefix"], D), dt)
    return x


def _block(seed, l):
    g, D, F, bf = _gen(seed, 100 + l), VIT["hidden"], VIT["ffn"], torch.bfloat16
    return {"ln1_g": _gain(g, D, bf), "ln1_b": _normal(g, (D,), bf, 0.1), "w_qkv": _normal(g, (3 * D, D), bf),
            "b_qkv": _normal(g, (3 * D,), bf), "w_o": _normal(g, (D, D), bf), "b_o": _normal(g, (D,), bf),
            "ln2_g": _gain(g, D, bf), "ln2_b": _normal(g, (D,), bf, 0.1), "w_fc1": _normal(g, (F, D), bf),
            "b_fc1": _normal(g, (F,), bf), "w_fc2": _normal(g, (D, F), bf), "b_fc2": _normal(g, (D,), bf)}


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "vision":
        cfg = B.make_vision_config(case["depth"], VIT["hidden"], VIT["heads"], VIT["hd"], VIT["ffn"],
                                   patch=VIT["patch"], merge=VIT["merge"], in_channels=VIT["channels"],
                                   out_hidden=VIT["out"], ln_eps=EPS, rope_theta=VIT_THETA, dtype=B.MTE_BF16,
                                   out_dtype=B.MTE_F32, max_images=case["images"],
                                   max_side=max(case["height"], case["width"]))
        enc = VisionEncoder(cfg, x["outer"], [_block(seed, l) for l in range(case["depth"])])
        return {"case": case, "enc": enc, "pixels": x["pixels"]}
    m, lens = _dims(case), _seq_lens(case["lens"])
    T, P = sum(lens), case["prefix"]
    cfg = B.make_config(case["layers"], m["hidden"], m["hq"], m["hkv"], m["hd"], m["ffn"], rms_eps=EPS,
                        rope_theta=THETA, mrope_section=m["sections"], mrope_layout=case["layout"],
                        qk_norm=case["qk_norm"], dtype=B.MTE_F32 if case["dtype"] == "f32" else B.MTE_BF16,
                        out_dtype=B.MTE_F32, max_tokens=max(T, P), max_batch=len(lens), max_seq=P + max(lens),
                        weight_format=B.MTE_WEIGHTS_E4M3 if case["weights"] == "e4m3" else B.MTE_WEIGHTS_DTYPE)
    enc = TextEncoder(cfg, [_layer(case, seed, l) for l in range(case["layers"])], x["final"])
    s = dict(x, case=case, enc=enc, lens=lens, layouts=[_layout(L) for L in lens])
    if case["kind"] == "layer":
        s["pos"] = build_positions(s["layouts"])
    elif case["kind"] == "prefixed":
        enc.reserve_prefix(P)
        s["prefix_pos"] = build_positions([(0, 0, 0, 0, P)])
        # the sequences' own positions go on after the prefix's
        s["pos"] = torch.cat([_positions([lay], P) for lay in s["layouts"]], 1).to(torch.int32).cuda()
    torch.cuda.synchronize()
    return s


def run(s):
    kind, enc = s["case"]["kind"], s["enc"]
    if kind == "vision":
        return enc.encode(s["pixels"])
    if kind == "layer":
        return enc.encode_layers(s["h"], s["pos"], s["lens"], 0, s["case"]["layers"])
    if kind == "prefixed":
        return enc.encode_prefixed(s["prefix"], s["prefix_pos"], s["embeds"], s["pos"], s["lens"])
    pos = build_positions(s["layouts"])
    return {"pos": pos, "hidden": enc.encode(s["embeds"], pos, s["lens"])}


# ------------------------------------------------- bytes, flops, tolerances
def work(case):
    """Each weight (at its stored width), input and output once; two flops per multiply-add of
    the products, attention over the visible keys only."""
    if case["kind"] == "vision":
        D, F, mm, kp = VIT["hidden"], VIT["ffn"], VIT["merge"] ** 2, VIT["channels"] * VIT["patch"] ** 2
        per = (case["height"] // VIT["patch"]) * (case["width"] // VIT["patch"])
        T = case["images"] * per
        block, tail = 4 * D * D + 2 * D * F, (mm * D) ** 2 + VIT["out"] * mm * D
        return {"bytes": 2 * (case["depth"] * block + kp * D + tail) + 2 * T * kp + 4 * (T // mm) * VIT["out"],
                "flops": 2 * T * (case["depth"] * block + kp * D) + 2 * (T // mm) * tail
                + case["depth"] * 4 * T * per * D}
    m, lens, P = _dims(case), _seq_lens(case["lens"]), case["prefix"]
    T, D, n = sum(lens), m["hidden"], case["layers"]
    par = D * (m["hq"] + 2 * m["hkv"]) * m["hd"] + m["hq"] * m["hd"] * D + 3 * D * m["ffn"]
    keys = sum(L * (L + 1) // 2 + L * P for L in lens) + P * (P + 1) // 2
    store = 4 if case["dtype"] == "f32" else 1 if case["weights"] == "e4m3" else 2
    io = 4 if case["kind"] == "layer" or case["dtype"] == "f32" else 2
    return {"bytes": n * par * store + (T + P) * (D * (io + 4) + 12),
            "flops": n * (2 * par * (T + P) + 4 * m["hq"] * m["hd"] * keys)}


def tolerance(case):
    """About four times the distance from exact() that one MI355X showed: relative errors of
    3.7e-7 (fp32, 2 layers), 2.5e-4 .. 3.2e-4 (one layer), 1.1e-3 (prefixed, 2 layers and the
    final norm), 3.6e-4 .. 4.3e-4 (vision, 1 to 3 blocks), 2.5e-3 (28 layers); the largest
    single differences are 15 to 20 times the relative error. Positions are exact."""
    if case["kind"] == "vision":
        rel = 1.7e-3
    elif case["dtype"] == "f32":
        rel = 2e-6
    else:
        rel = {"layer": 1.3e-3, "prefixed": 5e-3, "encode": 1e-2}[case["kind"]]
    return {"rel": rel, "max": 25 * rel}


# -------------------------------------------- the same in float64, plain torch
def _e4m3(w):
    """Rows as e4m3 values times the smallest power of two 2^e with max <= 448 * 2^e."""
    w = w.double()
    top = w.abs().amax(1, keepdim=True)
    f, e = torch.frexp(top)
    e = torch.where(f <= 0.875, e - 9, e - 8)
    scale = torch.where(top > 0, torch.ldexp(torch.ones_like(top), e), torch.ones_like(top))
    return (w / scale).float().to(torch.float8_e4m3fn).double() * scale


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g


def _rotate(z, ang):
    """z [T, H, d]; pair (j, j + d/2) turns by ang [T, d/2]."""
    h = z.shape[-1] // 2
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    u, w = z[..., :h], z[..., h:]
    return torch.cat([u * c - w * s, w * c + u * s], -1)


def _attend(q, k, v, causal, before=None):
    """One sequence: q [L, H, d], k / v [L, Hkv, d]; `before`: k, v of a prefix all see."""
    L, H, d = q.shape
    if before is not None:
        k, v = torch.cat([before[0], k]), torch.cat([before[1], v])
    k, v = (x.repeat_interleave(H // x.shape[1], 1).transpose(0, 1).contiguous() for x in (k, v))
    s = torch.matmul(q.transpose(0, 1).contiguous(), k.transpose(1, 2).contiguous()) / math.sqrt(d)
    if causal:
        i = torch.arange(L, device=q.device)[:, None] + k.shape[1] - L
        s = s.masked_fill(torch.arange(k.shape[1], device=q.device)[None] > i, -math.inf)
    return torch.matmul(torch.softmax(s, -1), v).transpose(0, 1)


def _decoder(case, seed, x, pos, lens, first=None):
    """All layers on the residual stream x [T, D] (float64); first: rows of a prefix sequence
    that every other sequence attends to."""
    m = _dims(case)
    hq, hkv, d, half = m["hq"], m["hkv"], m["hd"], m["hd"] // 2
    j = torch.arange(half, device="cuda")
    s = m["sections"]
    if case["layout"] == 0:
        ax = (j >= s[0]).long() + (j >= s[0] + s[1]).long()
    else:
        ax = torch.where((j % 3 == 1) & (j < 3 * s[1]), 1, torch.where((j % 3 == 2) & (j < 3 * s[2]), 2, 0))
    ang = pos.double()[ax].t() * torch.pow(torch.tensor(THETA, dtype=torch.float64, device="cuda"),
                                           -2.0 * j.double() / d)
    for l in range(case["layers"]):
        w = {k: v.double() if not (case["weights"] == "e4m3" and v.dim() == 2) else _e4m3(v)
             for k, v in _layer(case, seed, l).items()}
        a = _rms(x, w["attn_norm"])
        q, k, v = (torch.matmul(a, w[n].t()).reshape(-1, h, d) for n, h in (("w_q", hq), ("w_k", hkv), ("w_v", hkv)))
        if case["qk_norm"]:
            q, k = _rms(q, w["q_norm"]), _rms(k, w["k_norm"])
        q, k = _rotate(q, ang), _rotate(k, ang)
        o, at, before = [], 0, None
        for i, L in enumerate(lens):
            sl = slice(at, at + L)
            o.append(_attend(q[sl], k[sl], v[sl], True, before))
            if first and i == 0:
                before = (k[sl], v[sl])
            at += L
        x = x + torch.matmul(torch.cat(o).reshape(x.shape[0], hq * d), w["w_o"].t())
        a = _rms(x, w["mlp_norm"])
        x = x + torch.matmul(torch.nn.functional.silu(torch.matmul(a, w["w_gate"].t()))
                             * torch.matmul(a, w["w_up"].t()), w["w_down"].t())
    return x


def _ln(x, g, b):
    c = x - x.mean(-1, keepdim=True)
    return c / torch.sqrt((c * c).mean(-1, keepdim=True) + EPS) * g.double() + b.double()


def _gelu(z):
    return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))


def _tower(case, seed, x):
    n, p, mg, D, H, d = case["images"], VIT["patch"], VIT["merge"], VIT["hidden"], VIT["heads"], VIT["hd"]
    gh, gw = case["height"] // (p * mg), case["width"] // (p * mg)
    per = gh * gw * mg * mg
    o = {k: v.double() for k, v in x["outer"].items()}
    # [n, C, gh, mg, p, gw, mg, p] -> patches in merge-group order, (channel, row, column) vectors
    px = x["pixels"].double().reshape(n, VIT["channels"], gh, mg, p, gw, mg, p).permute(0, 2, 5, 3, 6, 1, 4, 7)
    h = torch.matmul(px.reshape(n * per, -1), o["patch_w"].t()) + o["patch_b"]
    grid = torch.arange(per, device="cuda")
    grp, inner = grid // (mg * mg), grid % (mg * mg)
    row, col = (grp // gw) * mg + inner // mg, (grp % gw) * mg + inner % mg
    j = torch.arange(d // 2, device="cuda")
    ang = torch.where(j[None] < d // 4, row[:, None], col[:, None]).double() * torch.pow(
        torch.tensor(VIT_THETA, dtype=torch.float64, device="cuda"), -2.0 * j.double() / d)
    for l in range(case["depth"]):
        w = {k: v.double() for k, v in _block(seed, l).items()}
        qkv = torch.matmul(_ln(h, w["ln1_g"], w["ln1_b"]), w["w_qkv"].t()) + w["b_qkv"]
        a = []
        for i in range(n):
            q, k, v = qkv[i * per:(i + 1) * per].reshape(per, 3, H, d).unbind(1)
            a.append(_attend(_rotate(q, ang), _rotate(k, ang), v, False))
        h = h + torch.matmul(torch.cat(a).reshape(n * per, D), w["w_o"].t()) + w["b_o"]
        z = _gelu(torch.matmul(_ln(h, w["ln2_g"], w["ln2_b"]), w["w_fc1"].t()) + w["b_fc1"])
        h = h + torch.matmul(z, w["w_fc2"].t()) + w["b_fc2"]
    u = _ln(h, o["merge_ln_g"], o["merge_ln_b"]).reshape(n * per // (mg * mg), -1)
    return torch.matmul(_gelu(torch.matmul(u, o["merge_w1"].t()) + o["merge_b1"]), o["merge_w2"].t()) + o["merge_b2"]


def exact(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "vision":
        return _tower(case, seed, x)
    lens = _seq_lens(case["lens"])
    layouts = [_layout(L) for L in lens]
    if case["kind"] == "prefixed":
        P = case["prefix"]
        pos = torch.cat([_positions([(0, 0, 0, 0, P)])] + [_positions([lay], P) for lay in layouts], 1).cuda()
        h = _decoder(case, seed, torch.cat([x["prefix"], x["embeds"]]).double(), pos, [P] + lens, first=True)
        h = _rms(h, x["final"].double())
        return h[:P], h[P:]
    pos = torch.cat([_positions([lay]) for lay in layouts], 1).cuda()
    if case["kind"] == "layer":
        return _decoder(case, seed, x["h"].double(), pos, lens)
    return {"pos": None, "hidden": _rms(_decoder(case, seed, x["embeds"].double(), pos, lens), x["final"].double())}
