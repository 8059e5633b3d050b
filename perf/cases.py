"""The work a program has this library do, as cases that can be measured: single steps of a decode or prompt pass, decoder layers,
and two whole calls, each through the package's public entry points.

A case is a dict of plain values; `kind` names the entry point.  Widths are those of the two models the benchmark
runs (hidden 4096 with 32 / 8 heads and inner size 14336; hidden 2048 with 16 / 4 heads, inner size 5632, 32000 tokens, 8 layers), or
multiples of 128 in between.  Weights are N(0, 0.02^2), activations and cache rows N(0, 1), norm weights N(1, 0.1^2)."""
import math
import random

import torch

import paper_2602_00182_amd as det
from paper_2602_00182_amd import decode

DEV = "cuda"
D = 128
EPS = 1e-5
SCALE = 0.08838834764831845  # 1/sqrt(128)
WIDE = dict(H=4096, Hq=32, Hkv=8, F=14336)
SMALL = dict(H=2048, Hq=16, Hkv=4, F=5632)
VOCAB, LAYERS = 32000, 8


def listed():
    return [
        # Picking the next tokens of a serving batch from its fp32 logits, with a seeded policy: the smallest call of a step.
        dict(name="draw-tokens", kind="sample", B=64, V=VOCAB, top_k=50),
        # The attention output projection of one interactive sequence: a launch of ten microseconds over 34 MB of weights.
        dict(name="out-proj-1", kind="proj", M=1, K=4096, N=4096),
        # The MLP's first projection, with its norm, for an ordinary serving batch whose size is no multiple of anything.
        dict(name="gate-up-45", kind="gateup", M=45, K=4096, F=14336),
        # The MLP's second projection for the largest decode batches: few columns, a long K, many rows.
        dict(name="down-proj-201", kind="proj", M=201, K=14336, N=4096),
        # The fused query/key/value projection of a prompt pass: norm, product, rotation and cache append of some thousand rows.
        dict(name="qkv-prompts", kind="qkv", H=4096, Hq=32, Hkv=8, prompts=5, longest=1000),
        # Attention of one sequence with a few thousand tokens behind it: all latency.
        dict(name="attn-1", kind="attn", B=1, Hq=32, Hkv=8, Lmax=4096, shortest=2900),
        # Attention of a serving batch whose sequences have run for different times.
        dict(name="attn-48-ragged", kind="attn", B=48, Hq=32, Hkv=8, Lmax=4096, shortest=200),
        # Causal attention of the prompts of a batch: every prompt token is a row that reads its own prefix.
        dict(name="attn-prompts", kind="attn_rows", Hq=32, Hkv=8, prompts=3, longest=2000),
        # One decoder layer of a serving batch at a context of about two thousand.
        dict(name="layer-32", kind="layer", quantized=False, prompts=0, B=32, Lmax=2048, **WIDE),
        # The same layer with quantized projections for one sequence: the case quantization is chosen for.
        dict(name="qlayer-1", kind="layer", quantized=True, prompts=0, B=1, Lmax=2048, **WIDE),
        # A quantized layer of the small model over the prompts of a batch.
        dict(name="qlayer-prompts", kind="layer", quantized=True, prompts=6, B=512, Lmax=512, **SMALL),
        # A whole job of the small model: prompts of 16..512 tokens in one pass, then greedy tokens, the logits kept for the commitment.
        dict(name="job-24", kind="job", quantized=False, prompts=24, longest=512, new=24),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    return 128 * _log(rng, lo // 128, hi // 128)


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["sample", "proj", "proj", "gateup", "gateup", "qkv", "attn", "attn", "attn_rows", "layer", "layer", "layer_rows", "job"])
    heads = rng.choice([(32, 8), (16, 4), (16, 16), (16, 2)])
    if kind == "sample":  # top_k 1 is the greedy choice
        return dict(kind=kind, B=_log(rng, 1, 64), V=rng.choice([VOCAB, _log(rng, 8000, 60000)]), top_k=_log(rng, 1, 1000))
    if kind == "proj":
        K, N = rng.choice([(4096, 4096), (14336, 4096), (2048, 2048), (5632, 2048), (_width(rng, 2048, 14336), _width(rng, 2048, 14336))])
        return dict(kind=kind, M=_log(rng, 1, 4096), K=K, N=N)
    if kind == "gateup":
        K, F = rng.choice([(4096, 14336), (2048, 5632), (_width(rng, 2048, 4096), _width(rng, 4096, 14336))])
        return dict(kind=kind, M=_log(rng, 1, 4096), K=K, F=F)
    if kind == "qkv":
        return dict(kind=kind, H=128 * heads[0], Hq=heads[0], Hkv=heads[1], prompts=_log(rng, 1, 16), longest=_log(rng, 16, 1000))
    if kind == "attn":
        B = _log(rng, 1, 64)
        Lmax = _log(rng, 300, min(32768, 4096 * 64 // B))
        return dict(kind=kind, B=B, Hq=heads[0], Hkv=heads[1], Lmax=Lmax, shortest=rng.randint(1, Lmax))
    if kind == "attn_rows":
        prompts = _log(rng, 1, 12)
        return dict(kind=kind, Hq=heads[0], Hkv=heads[1], prompts=prompts, longest=_log(rng, 40, min(4000, 12000 // prompts)))
    if kind == "job":
        return dict(kind=kind, quantized=rng.random() < 0.5, prompts=_log(rng, 1, 24), longest=_log(rng, 40, 512), new=_log(rng, 2, 24))
    size = rng.choice([WIDE, SMALL])
    quantized = rng.random() < 0.5
    if kind == "layer":
        return dict(kind="layer", quantized=quantized, prompts=0, B=_log(rng, 1, 128), Lmax=_log(rng, 200, 2500), **size)
    longest = _log(rng, 40, 1000)
    return dict(kind="layer", quantized=quantized, prompts=_log(rng, 1, 8), B=longest, Lmax=longest, **size)


# ------------------------------------------------------------------------------------------------ inputs


def _lengths(n, lo, hi):
    """n lengths in lo..hi, the same for every seed of a case; the longest is hi."""
    r = random.Random(n * 1000003 + hi)
    return [hi] + [r.randint(lo, hi) for _ in range(n - 1)]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, shape, std=1.0, mean=0.0):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(mean, std, generator=g)


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device=DEV)


def _rope(Lmax):
    inv = 5.0e5 ** (-torch.arange(D // 2, dtype=torch.float64, device=DEV) * 2 / D)
    a = torch.arange(Lmax, dtype=torch.float64, device=DEV)[:, None] * inv[None, :]
    return a.cos().float().contiguous(), a.sin().float().contiguous()


def _rows(lens):
    """Positions, slots and lengths of the rows of prompts that go through in one call."""
    pos = [p for n in lens for p in range(n)]
    slot = [s for s, n in enumerate(lens) for _ in range(n)]
    return _i32(pos), _i32(slot), _i32([p + 1 for p in pos])


def _layer_rows(c):
    """(lengths, rows) of a layer case: prompts in one pass, or one new token of each of B sequences."""
    if c["prompts"]:
        lens = _lengths(c["prompts"], max(1, c["B"] // 4), c["B"])
        return lens, sum(lens)
    return _lengths(c["B"], c["Lmax"] // 2, c["Lmax"]), c["B"]


def _layer_raw(g, c):
    H, Hq, Hkv, F = c["H"], c["Hq"], c["Hkv"], c["F"]
    return dict(norm1=_normal(g, (H,), 0.1, 1.0), wqkv=_normal(g, (H, (Hq + 2 * Hkv) * D), 0.02), wo=_normal(g, (Hq * D, H), 0.02),
                norm2=_normal(g, (H,), 0.1, 1.0), wgu=_normal(g, (H, 2 * F), 0.02), wdown=_normal(g, (F, H), 0.02))


def _model_raw(g):
    w = dict(embed=_normal(g, (VOCAB, SMALL["H"])), final_norm=_normal(g, (SMALL["H"],), 0.1, 1.0), lm_head=_normal(g, (SMALL["H"], VOCAB), 0.02))
    w["layers"] = [_layer_raw(g, SMALL) for _ in range(LAYERS)]
    return w


def _inputs(c, seed):
    """The tensors a case computes from, as plain row-major ones."""
    g, kind = _gen(seed), c["kind"]
    s = {}
    if kind == "sample":
        s["logits"] = torch.empty((c["B"], c["V"]), device=DEV).normal_(0, 2.5, generator=g)
    elif kind == "proj":
        s.update(a=_normal(g, (c["M"], c["K"])), w=_normal(g, (c["K"], c["N"]), 0.02), r=_normal(g, (c["M"], c["N"])))
    elif kind == "gateup":
        s.update(x=_normal(g, (c["M"], c["K"])), wn=_normal(g, (c["K"],), 0.1, 1.0), w=_normal(g, (c["K"], 2 * c["F"]), 0.02))
    elif kind == "qkv":
        lens = _lengths(c["prompts"], max(1, c["longest"] // 4), c["longest"])
        s.update(x=_normal(g, (sum(lens), c["H"])), wn=_normal(g, (c["H"],), 0.1, 1.0), w=_normal(g, (c["H"], (c["Hq"] + 2 * c["Hkv"]) * D), 0.02))
        s["pos"], s["slots"], _ = _rows(lens)
        s["cache"] = (len(lens), c["Hkv"], c["longest"], D)
    elif kind in ("attn", "attn_rows"):
        if kind == "attn":
            lens = _lengths(c["B"], c["shortest"], c["Lmax"])
            s.update(lens=_i32(lens), q=_normal(g, (c["B"], c["Hq"], D)))
            shape = (c["B"], c["Hkv"], c["Lmax"], D)
        else:
            lens = _lengths(c["prompts"], max(1, c["longest"] // 4), c["longest"])
            _, s["slots"], s["lens"] = _rows(lens)
            s["q"] = _normal(g, (sum(lens), c["Hq"], D))
            shape = (c["prompts"], c["Hkv"], c["longest"], D)
        s.update(k=_normal(g, shape), v=_normal(g, shape))
    elif kind == "layer":
        lens, R = _layer_rows(c)
        shape = (len(lens), c["Hkv"], c["Lmax"], D)
        s.update(raw=_layer_raw(g, c), x0=_normal(g, (R, c["H"])), k=_normal(g, shape), v=_normal(g, shape))
        if c["prompts"]:
            s["pos"], s["slots"], _ = _rows(lens)
        else:
            s.update(pos=_i32([n - 1 for n in lens]), slots=None)
    elif kind == "job":
        lens = _lengths(c["prompts"], min(16, c["longest"]), c["longest"])
        s.update(raw=_model_raw(g), lens=torch.tensor(lens, dtype=torch.int32, device=DEV))
        s["prompts"] = torch.randint(0, VOCAB, (len(lens), c["longest"]), generator=g, device=DEV, dtype=torch.int32)
    return s


def _empty(shape, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _layer_struct(raw, c, quantized):
    pack = det.quant_pack_weight if quantized else det.pack_weight
    gu = det.quant_pack_gate_up if quantized else det.pack_gate_up
    qkv = det.quant_pack_qkv if quantized else det.pack_qkv
    return det.layer_weights(raw["norm1"], qkv(raw["wqkv"], c["Hq"], c["Hkv"], D), pack(raw["wo"]), raw["norm2"], gu(raw["wgu"]), pack(raw["wdown"]))


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(c, seed)
    s["case"] = c
    if kind == "sample":
        s.update(ids=torch.arange(c["B"], dtype=torch.int32, device=DEV), steps=torch.full((c["B"],), 17, dtype=torch.int32, device=DEV), out=_empty((c["B"],), torch.int32))
    elif kind == "proj":
        s.update(wp=det.pack_weight(s.pop("w")), out=_empty((c["M"], c["N"])))
    elif kind == "gateup":
        s.update(wp=det.pack_gate_up(s.pop("w")), h=_empty((c["M"], c["K"])), out=_empty((c["M"], c["F"])))
    elif kind == "qkv":
        M, shape = s["x"].shape[0], s["cache"]
        s.update(wp=det.pack_qkv(s.pop("w"), c["Hq"], c["Hkv"], D), h=_empty((M, c["H"])), out=_empty((M, c["Hq"], D)))
        s.update(k=torch.zeros(shape, dtype=torch.bfloat16, device=DEV), v=torch.zeros(shape, dtype=torch.bfloat16, device=DEV))
        s["cos"], s["sin"] = _rope(c["longest"])
    elif kind in ("attn", "attn_rows"):
        s["out"] = torch.empty_like(s["q"])
        s["ws"] = _empty((det.det_attn_decode_workspace_bytes(s["q"].shape[0], c["Hq"], D, s["k"].shape[2]),), torch.uint8)
    elif kind == "layer":
        s["w"] = _layer_struct(s.pop("raw"), c, c["quantized"])
        s["cfg"] = det.layer_cfg(c["H"], c["Hq"], c["Hkv"], D, c["F"], c["Lmax"], EPS, SCALE)
        s["x"] = torch.empty_like(s["x0"])
        need = det.det_qdecoder_layer_workspace_bytes if c["quantized"] else det.det_decoder_layer_workspace_bytes
        s["ws"] = _empty((need(s["cfg"], s["x"].shape[0]),), torch.uint8)
        s["cos"], s["sin"] = _rope(c["Lmax"])
    elif kind == "job":
        cfg = decode.ModelCfg(SMALL["H"], SMALL["Hq"], SMALL["Hkv"], D, SMALL["F"], VOCAB, LAYERS, EPS, SCALE)
        s["model"] = decode.DecodeModel(cfg, s.pop("raw"), quantized=c["quantized"])
        s["cos"], s["sin"] = _rope(c["longest"] + c["new"])
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "sample":
        if c["top_k"] == 1:
            det.det_argmax(s["logits"], s["out"])
        else:
            det.det_sample(s["logits"], 0.8, c["top_k"], 0.95, 1234, s["ids"], s["steps"], s["out"])
        return s["out"]
    if kind == "proj":
        det.det_gemm_bf16_residual(s["a"], s["wp"], s["r"], s["out"], c["N"], c["K"])
        return s["out"]
    if kind == "gateup":
        det.det_rmsnorm_gemm_swiglu_bf16(s["x"], s["wn"], EPS, s["wp"], s["h"], s["out"], c["F"])
        return s["out"]
    if kind == "qkv":
        det.det_rmsnorm_gemm_qkv_rope_append(s["x"], s["wn"], EPS, s["wp"], s["h"], s["out"], s["k"], s["v"], s["pos"], s["slots"], s["cos"], s["sin"])
        return s["out"], s["k"], s["v"]
    if kind == "attn":
        det.det_attn_decode(s["q"], s["k"], s["v"], s["lens"], s["out"], s["ws"], SCALE)
        return s["out"]
    if kind == "attn_rows":
        det.det_attn_decode_rows(s["q"], s["k"], s["v"], s["lens"], s["slots"], s["out"], s["ws"], SCALE)
        return s["out"]
    if kind == "layer":
        s["x"].copy_(s["x0"])  # the layer works in place
        if c["quantized"]:
            det.det_qdecoder_layer(s["w"], s["cfg"], s["x"], s["k"], s["v"], s["pos"], s["slots"], s["cos"], s["sin"], s["ws"])
        elif s["slots"] is None:
            det.det_decoder_layer(s["w"], s["cfg"], s["x"], s["k"], s["v"], s["pos"], s["cos"], s["sin"], s["ws"])
        else:
            det.det_decoder_layer_rows(s["w"], s["cfg"], s["x"], s["k"], s["v"], s["pos"], s["slots"], s["cos"], s["sin"], s["ws"])
        return s["x"], s["k"], s["v"]
    tokens, logits = decode.prefill_decode(s["model"], s["prompts"], s["lens"], c["new"], s["cos"], s["sin"], keep_logits=True)
    return tokens, logits


# ------------------------------------------------------------------------------------------------ what a pass cannot do without


def _attn_work(Hq, Hkv, lens, causal):
    """Bytes of the keys and values read once, and operations of the scores and the weighted sums."""
    pairs = sum(n * (n + 1) // 2 if causal else n for n in lens)
    return 4 * D * Hkv * sum(lens), 4 * D * Hq * pairs


def _layer_work(c, lens, rows, causal, quantized):
    H, Hq, Hkv, F = c["H"], c["Hq"], c["Hkv"], c["F"]
    weights = H * (Hq + 2 * Hkv) * D + Hq * D * H + 3 * H * F
    b, f = _attn_work(Hq, Hkv, lens, causal)
    return weights * (4.25 / 8 if quantized else 2) + b + 4 * rows * H, 2 * rows * weights + f


def work(case):
    c, kind = case, case["kind"]
    if kind == "sample":
        b, f = 4 * c["B"] * c["V"], c["B"] * c["V"]
    elif kind == "proj":
        M, K, N = c["M"], c["K"], c["N"]
        b, f = 2 * (K * N + M * K + 2 * M * N), 2 * M * K * N
    elif kind == "gateup":
        M, K, F = c["M"], c["K"], c["F"]
        b, f = 2 * (2 * K * F + M * K + M * F), 4 * M * K * F
    elif kind == "qkv":
        M, N = sum(_lengths(c["prompts"], max(1, c["longest"] // 4), c["longest"])), (c["Hq"] + 2 * c["Hkv"]) * D
        b, f = 2 * (c["H"] * N + M * c["H"] + M * N), 2 * M * c["H"] * N
    elif kind == "attn":
        lens = _lengths(c["B"], c["shortest"], c["Lmax"])
        b, f = _attn_work(c["Hq"], c["Hkv"], lens, False)
        b += 4 * c["B"] * c["Hq"] * D
    elif kind == "attn_rows":
        lens = _lengths(c["prompts"], max(1, c["longest"] // 4), c["longest"])
        b, f = _attn_work(c["Hq"], c["Hkv"], lens, True)
        b += 4 * sum(lens) * c["Hq"] * D
    elif kind == "layer":
        lens, R = _layer_rows(c)
        b, f = _layer_work(c, lens, R, bool(c["prompts"]), c["quantized"])
    else:
        lens = _lengths(c["prompts"], min(16, c["longest"]), c["longest"])
        B, H = len(lens), SMALL["H"]
        b = f = 0
        for step in range(c["new"]):
            now = lens if step == 0 else [n + step for n in lens]
            lb, lf = _layer_work(SMALL, now, sum(lens) if step == 0 else B, step == 0, c["quantized"])
            b += LAYERS * lb + H * VOCAB * (4.25 / 8 if c["quantized"] else 2) + 4 * B * VOCAB
            f += LAYERS * lf + 2 * B * H * VOCAB
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Four times the distance from the 64-bit result that was measured, which is bf16 rounding: once where only the output is
    rounded, several times where normalized rows, projections and activations are rounded (or quantized) on the way."""
    kind = case["kind"]
    if kind == "sample":
        return "exact"
    if kind in ("layer", "job"):
        rel = 3e-2 if kind == "job" or case["quantized"] else 2e-2
    else:
        rel = {"proj": 9e-3, "gateup": 1.6e-2, "qkv": 1.2e-2, "attn": 7e-3, "attn_rows": 7e-3}[kind]
    return {"rel": rel, "max": 10 * rel}


# ------------------------------------------------------------------------------------------------ the same in 64 bits


def _norm64(x, w):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * w.double()


def _quant_w(w):
    """The weight the 4-bit format holds: blocks of 64 along K, scale amax/7 rounded to bf16."""
    b = w.float().reshape(-1, 64, w.shape[1])
    s = (b.abs().amax(1, keepdim=True) / 7).to(torch.bfloat16).float()
    q = torch.where(s == 0, torch.zeros_like(b), (b / s).round().clamp(-8, 7))
    return (q.double() * s.double()).reshape(w.shape)


def _quant_a(a):
    """The activations the 8-bit format holds: blocks of 64 along K, scale amax/127."""
    b = a.to(torch.bfloat16).float().reshape(a.shape[0], -1, 64)
    s = b.abs().amax(2, keepdim=True) / 127
    q = torch.where(s == 0, torch.zeros_like(b), (b / s).round().clamp(-127, 127))
    return (q.double() * s.double()).reshape(a.shape)


def _product64(a, w, quantized):
    if quantized:
        return torch.cat([_quant_a(r) for r in a.split(1024)]) @ _quant_w(w)
    return a @ w.double()


def _rotate64(x, pos, cos, sin):
    lo, hi = x[..., : D // 2], x[..., D // 2:]
    co, si = cos.double()[pos.long()][:, None, :], sin.double()[pos.long()][:, None, :]
    return torch.cat([lo * co - hi * si, lo * si + hi * co], -1)


def _attend64(q, k, v, lens, slots):
    """q [R, Hq, D]; row r reads the first lens[r] rows of slot slots[r] of k, v [S, Hkv, Lmax, D]."""
    R, Hq, _ = q.shape
    Hkv = k.shape[1]
    out = torch.zeros_like(q)
    for s in slots.unique().tolist():
        at = (slots == s).nonzero()[:, 0]
        for part in at.split(512):
            n = int(lens[part].max())
            if n == 0:
                continue
            qs = q[part].reshape(len(part), Hkv, Hq // Hkv, D).permute(1, 0, 2, 3).reshape(Hkv, -1, D)
            kt = k[s, :, :n].double().transpose(1, 2).contiguous()
            scores = (qs @ kt).reshape(Hkv, len(part), Hq // Hkv, n) * SCALE
            dead = torch.arange(n, device=q.device)[None, :] >= lens[part].long()[:, None]
            scores.masked_fill_(dead[None, :, None, :], -math.inf)
            p = torch.softmax(scores, -1).nan_to_num(0).reshape(Hkv, -1, n)
            o = (p @ v[s, :, :n].double().contiguous()).reshape(Hkv, len(part), Hq // Hkv, D)
            out[part] = o.permute(1, 0, 2, 3).reshape(len(part), Hq, D)
    return out


def _layer64(x, raw, c, k, v, pos, slots, cos, sin, quantized):
    """One decoder layer on rows x (float64); k and v (float64) take the new rows."""
    R, Hq, Hkv, F = x.shape[0], c["Hq"], c["Hkv"], c["F"]
    qkv = _product64(_norm64(x, raw["norm1"]), raw["wqkv"], quantized).reshape(R, Hq + 2 * Hkv, D)
    q = _rotate64(qkv[:, :Hq], pos, cos, sin)
    k[slots.long(), :, pos.long()] = _rotate64(qkv[:, Hq:Hq + Hkv], pos, cos, sin)
    v[slots.long(), :, pos.long()] = qkv[:, Hq + Hkv:]
    x = x + _product64(_attend64(q, k, v, pos + 1, slots).reshape(R, Hq * D), raw["wo"], quantized)
    gu = _product64(_norm64(x, raw["norm2"]), raw["wgu"], quantized)
    m = torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]
    return x + _product64(m, raw["wdown"], quantized)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "sample":
        return None
    s = _inputs(c, seed)
    if kind == "proj":
        return s["a"].double() @ s["w"].double() + s["r"].double()
    if kind == "gateup":
        gu = _norm64(s["x"].double(), s["wn"]) @ s["w"].double()
        return torch.nn.functional.silu(gu[:, :c["F"]]) * gu[:, c["F"]:]
    if kind == "qkv":
        cos, sin = _rope(c["longest"])
        R, Hq, Hkv = s["x"].shape[0], c["Hq"], c["Hkv"]
        qkv = (_norm64(s["x"].double(), s["wn"]) @ s["w"].double()).reshape(R, Hq + 2 * Hkv, D)
        k, v = torch.zeros(s["cache"], dtype=torch.float64, device=DEV), torch.zeros(s["cache"], dtype=torch.float64, device=DEV)
        k[s["slots"].long(), :, s["pos"].long()] = _rotate64(qkv[:, Hq:Hq + Hkv], s["pos"], cos, sin)
        v[s["slots"].long(), :, s["pos"].long()] = qkv[:, Hq + Hkv:]
        return _rotate64(qkv[:, :Hq], s["pos"], cos, sin), k, v
    if kind in ("attn", "attn_rows"):
        slots = s.get("slots")
        slots = torch.arange(c["B"], device=DEV) if slots is None else slots
        return _attend64(s["q"].double(), s["k"], s["v"], s["lens"], slots)
    if kind == "layer":
        cos, sin = _rope(c["Lmax"])
        slots = torch.arange(c["B"], device=DEV) if s["slots"] is None else s["slots"]
        k, v = s["k"].double(), s["v"].double()
        x = _layer64(s["x0"].double(), s["raw"], c, k, v, s["pos"], slots, cos, sin, c["quantized"])
        return x, k, v
    # the job: the logits of its first step, which follow from the prompts alone
    lens, cos_sin = s["lens"].tolist(), _rope(c["longest"] + c["new"])
    pos, slots, _ = _rows(lens)
    raw = s["raw"]
    x = raw["embed"][s["prompts"][slots.long(), pos.long()].long()].double()
    shape = (len(lens), SMALL["Hkv"], c["longest"], D)
    for lw in raw["layers"]:
        k, v = torch.zeros(shape, dtype=torch.float64, device=DEV), torch.zeros(shape, dtype=torch.float64, device=DEV)
        x = _layer64(x, lw, SMALL, k, v, pos, slots, *cos_sin, c["quantized"])
    last = torch.tensor(lens, device=DEV).cumsum(0) - 1
    first = _product64(_norm64(x[last], raw["final_norm"]), raw["lm_head"], c["quantized"])
    return None, [first] + [None] * (c["new"] - 1)
