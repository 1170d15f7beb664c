"""The workloads this library's speed is judged on, through the entry points a serving engine or a calibration job calls.

A case is one call (or one decode step) of one decoder layer:

* "step"      one decode step: the cache write of the current tokens, then the decode (int2kv_append_decode);
* "decode"    the decode alone over an INT2 cache (int2kv_decode);
* "window"    the decode with BF16 sink and recent windows (int2kv_decode_window);
* "append"    the cache write of a prompt (int2kv_quantize_append, or int2kv_quantize_append_rope for pre-RoPE keys and
              the Hadamard rotation);
* "outerr"    the output-error diagnostics (int2kv_output_error);
* "calibrate" OptR's offline calibration (int2kv_optr_calibrate).

Caches hold group-quantized N(0, 1) rows (centered keys and values in their rotated bases), written here with plain torch
in the documented record layout, so that `exact` needs nothing of the library. Weights, plans, workspaces and output
buffers are made once in `prepare`, as a serving loop keeps them. Everything but the context lengths (a property of the
case) is drawn from the seed.
"""
import math
import random

import numpy as np
import torch

from paper_2608_02691_amd import int2kv as K

D = 128         # head dimension
PAGE = 16       # tokens of a cache block
THETA = 1.0e6   # RoPE base
SCALE = 1.0 / math.sqrt(D)


def _case(name, kind, **kw):
    base = {
        "step": dict(batch=1, ctx_lo=256, ctx_hi=256, q_heads=32, kv_heads=8, group=32, d_model=0, wo="none"),
        "decode": dict(batch=1, ctx_lo=256, ctx_hi=256, q_heads=32, kv_heads=8, group=32, d_model=0, wo="none"),
        "window": dict(batch=1, ctx_lo=256, ctx_hi=256, q_heads=32, kv_heads=8, group=128, d_model=0, wo="none",
                       sink=64, recent=256),
        "append": dict(tokens=1, kv_heads=8, group=32, rope=False, hadamard=False, clip_k=1.0, clip_v=1.0),
        "outerr": dict(batch=1, ctx_lo=256, ctx_hi=256, q_heads=32, kv_heads=8, group=32, d_model=4096, dy=False),
        "calibrate": dict(q_heads=32, kv_heads=8, d_model=4096, group=128, calib_seqs=7, calib_lo=328, calib_hi=560,
                          held_seqs=6, held_lo=400, held_hi=640, sink=64, recent=256, steps=20, eval_every=10),
    }[kind]
    return {"name": name, "kind": kind, **base, **kw} if name else {"kind": kind, **base, **kw}


def listed():
    return [
        # the smallest call: one short sequence, one head; launches and latencies are all of it
        _case("step-b1-tiny", "step", ctx_lo=256, ctx_hi=256, q_heads=1, kv_heads=1),
        # a single user's chat, one Qwen3-8B-shaped layer, at an odd context, with the layer's output projection
        _case("step-b1-1k", "step", ctx_lo=1011, ctx_hi=1011, d_model=4096, wo="prepared_folded"),
        # a small serving batch of the same layer: 16 sequences of 4K tokens
        _case("step-b16-4k", "step", batch=16, ctx_lo=4096, ctx_hi=4096, d_model=4096, wo="prepared_folded"),
        # long-context question answering: one sequence of 128K tokens, attention output only
        _case("decode-b1-128k", "decode", ctx_lo=131072, ctx_hi=131072),
        # a full ragged serving batch (the largest case): 64 sequences of 512 to 32K tokens, 40/8 heads
        _case("step-ragged64", "step", batch=64, ctx_lo=512, ctx_hi=32768, q_heads=40, d_model=5120,
              wo="prepared_folded"),
        # the paper's serving setting: 128-channel groups and BF16 windows of 64 + 256 tokens beside the cache
        _case("window-ragged32-g128", "window", batch=32, ctx_lo=512, ctx_hi=16384, q_heads=40, d_model=5120,
              wo="prepared_folded"),
        # weights as the model holds them (row-major bf16, no set-up), eight query heads per KV head, ragged short contexts
        _case("decode-b8-gq8-plain", "decode", batch=8, ctx_lo=37, ctx_hi=2500, kv_heads=4, d_model=4096, wo="plain"),
        # prefill of four 8K prompts: the large cache write
        _case("append-32k", "append", tokens=32768),
        # prefill of one 2K prompt in the paper's serving setting, fused with RoPE (keys arrive pre-RoPE)
        _case("append-2k-rope-g128", "append", tokens=2011, group=128, rope=True, clip_k=0.96, clip_v=0.92),
        # a large prefill with RoPE and the Hadamard base rotation that OptR refines
        _case("append-16k-rope-had", "append", tokens=16384, rope=True, hadamard=True),
        # output-error diagnostics of a cache against its full-precision rows
        _case("outerr-b16-4k", "outerr", batch=16, ctx_lo=4096, ctx_hi=4096),
        # calibration of one layer's eight KV heads at the paper's settings, 20 steps for keys and 20 for values
        _case("calibrate-1-layer", "calibrate"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "decode", "window", "append", "append", "outerr", "calibrate"])
    group = rng.choice([32, 128])
    if kind in ("step", "decode", "window"):
        q_heads, kv_heads = rng.choice([(32, 8), (40, 8), (32, 4), (16, 8), (4, 1)])
        batch = _log_int(rng, 1, 64)
        hi = min(_log_int(rng, 64, 131072 if batch == 1 else 32768), 1_600_000 // batch)
        lo = max(1, int(hi * rng.choice([1.0, 0.5, 0.02])))
        wo = rng.choice(["none", "plain", "folded", "prepared", "prepared_folded"])
        kw = dict(batch=batch, ctx_lo=lo, ctx_hi=hi, q_heads=q_heads, kv_heads=kv_heads, group=group, wo=wo,
                  d_model=0 if wo == "none" else rng.choice([4096, 5120]))
        if kind == "window":
            kw.update(sink=rng.choice([0, 16, 64]), recent=rng.randint(1, 256))
        return _case("", kind, **kw)
    if kind == "append":
        clip_k, clip_v = rng.choice([(1.0, 1.0), (0.96, 0.92)])
        return _case("", kind, tokens=_log_int(rng, 1, 32768), kv_heads=rng.choice([8, 8, 4, 1]), group=group,
                     rope=rng.random() < 0.5, hadamard=rng.random() < 0.3, clip_k=clip_k, clip_v=clip_v)
    if kind == "outerr":
        hi = _log_int(rng, 128, 4096)
        return _case("", kind, batch=_log_int(rng, 1, 16), ctx_lo=max(1, int(hi * rng.choice([1.0, 0.3]))), ctx_hi=hi,
                     q_heads=rng.choice([32, 16]), group=group, dy=rng.random() < 0.3)
    heads = rng.choice([1, 2, 8])
    window = rng.choice([(64, 256), (0, 0)])
    steps = rng.randint(4, 16)
    return _case("", kind, kv_heads=heads, q_heads=heads * rng.choice([1, 4]), group=group, calib_seqs=rng.randint(2, 6),
                 calib_lo=rng.randint(130, 330), held_seqs=rng.randint(1, 5), held_lo=rng.randint(200, 400),
                 held_hi=560, sink=window[0], recent=window[1], steps=steps, eval_every=rng.randint(2, steps))


# ---------------------------------------------------------------------------------------------
# Inputs

def _lens(case):
    """Context lengths: a property of the case, the same for every seed."""
    lo, hi = case["ctx_lo"], case["ctx_hi"]
    r = random.Random("%d %d %d" % (case["batch"], lo, hi))
    return [r.randint(lo, hi) for _ in range(case["batch"])]


def _gen(seed, salt):
    return torch.Generator("cuda").manual_seed(int(seed) * 64 + salt)


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _rotations(seed, heads):
    """Haar-random orthogonal matrices, fp32 [heads, 128, 128]: QR of a Gaussian with the signs of diag(R) folded in."""
    g = torch.Generator().manual_seed(int(seed))
    q, r = torch.linalg.qr(torch.randn((heads, D, D), generator=g, dtype=torch.float64))
    return (q * torch.sign(torch.diagonal(r, dim1=1, dim2=2))[:, None, :]).float().contiguous().cuda()


def _offsets(seed, heads):
    """Constant key offsets: three channels per KV head at 10 to 30 (what key centering removes)."""
    r = random.Random(int(seed))
    off = torch.zeros((heads, D))
    for h in range(heads):
        for c in r.sample(range(D), 3):
            off[h, c] = r.uniform(10.0, 30.0)
    return off.cuda()


def _quantize(x, group, clip=1.0):
    """Group-wise affine INT2 of fp32 rows [..., 128]: codes (uint8 [..., 128]), fp16 scale and zero [..., 128 / group]."""
    g = x.reshape(x.shape[:-1] + (D // group, group))
    mn, mx = g.amin(-1), g.amax(-1)
    if clip != 1.0:
        c = torch.tensor(clip, dtype=torch.float32, device=x.device)
        mn, mx = c * mn, c * mx
    s, z = ((mx - mn) / torch.full_like(mx, 3.0)).half(), mn.half()  # a true division: by a scalar it is a product
    sf, zf = s.float()[..., None], z.float()[..., None]
    inv = torch.where(sf > 0, 1.0 / sf, torch.zeros_like(sf))
    codes = torch.clamp(torch.round((g - zf) * inv), 0, 3).to(torch.uint8)
    return codes.reshape(x.shape), s, z


def _dequantize(codes, s, z, group):
    g = codes.double().reshape(codes.shape[:-1] + (D // group, group))
    return (g * s.double()[..., None] + z.double()[..., None]).reshape(codes.shape)


def _halves(codes):
    """16-bit halves of the packed codes: half m holds channel 16 p + m at bits 2 p."""
    c = codes.reshape(codes.shape[:-1] + (8, 16)).to(torch.int32)
    half = c[..., 0, :].clone()
    for p in range(1, 8):
        half += c[..., p, :] << (2 * p)
    return half.to(torch.int16)


def _records(k_rows, v_rows, group):
    """Packed records uint8 [n, H, bytes] of n blocks of 16 rows: k_rows, v_rows fp32 [n, 16, H, 128]."""
    n, _, H, _ = k_rows.shape
    flat = lambda t: t.contiguous().view(torch.uint8).reshape(n, H, -1)  # noqa: E731
    kc, ks, kz = _quantize(k_rows.transpose(1, 2), group)
    vc, vs, vz = _quantize(v_rows.transpose(1, 2), group)
    return torch.cat([flat(_halves(kc)), flat(_halves(vc).transpose(2, 3)), flat(torch.stack([ks, kz], -1)),
                      flat(vs.transpose(2, 3)), flat(vz.transpose(2, 3))], dim=-1)


def _rows_of(records, group):
    """Dequantized rows fp64 [n, 16, H, 128] (keys, values) of packed records [n, H, bytes]."""
    n, H, _ = records.shape
    ng = D // group
    u16 = lambda t: t.contiguous().view(torch.int16).to(torch.int32) & 0xFFFF  # noqa: E731
    shift = 2 * torch.arange(8, device=records.device, dtype=torch.int32)
    codes = lambda h: ((h[..., None, :] >> shift[:, None]) & 3).reshape(h.shape[:-1] + (D,))  # noqa: E731
    kh = u16(records[..., :512]).reshape(n, H, PAGE, 16)
    vh = u16(records[..., 512:1024]).reshape(n, H, 16, PAGE).transpose(2, 3)
    km = records[..., 1024:1024 + 64 * ng].contiguous().view(torch.float16).reshape(n, H, PAGE, ng, 2)
    vm = records[..., 1024 + 64 * ng:].contiguous().view(torch.float16).reshape(n, H, 2, ng, PAGE).transpose(3, 4)
    k = _dequantize(codes(kh), km[..., 0], km[..., 1], group)
    v = _dequantize(codes(vh), vm[:, :, 0], vm[:, :, 1], group)
    return k.transpose(1, 2), v.transpose(1, 2)


def _paging(seed, lens):
    """Block table of the sequences over a permuted pool: (table int32 [B, max blocks], pages per sequence, blocks)."""
    pages = [(n + PAGE - 1) // PAGE for n in lens]
    total = sum(pages)
    phys = torch.randperm(total, generator=torch.Generator().manual_seed(int(seed))).to(torch.int32)
    table = torch.zeros((len(lens), max(pages)), dtype=torch.int32)
    at = 0
    for b, n in enumerate(pages):
        table[b, :n] = phys[at:at + n]
        at += n
    return table, pages, phys


def _random_pool(seed, phys, heads, group):
    """A cache of group-quantized N(0, 1) rows for every physical block."""
    pool = torch.empty((len(phys), heads, K.RECORD_BYTES_BY_GROUP[group]), dtype=torch.uint8, device="cuda")
    g, phys, chunk = _gen(seed, 1), phys.cuda().long(), max(1, 32768 // heads)
    for i in range(0, len(phys), chunk):
        at = phys[i:i + chunk]
        pool[at] = _records(_randn(g, len(at), PAGE, heads, D), _randn(g, len(at), PAGE, heads, D), group)
    return pool


def _weights(seed, d_model, q_heads):
    return (_randn(_gen(seed, 2), d_model, q_heads * D) / math.sqrt(d_model)).to(torch.bfloat16)


def _bf16(x):
    return x.to(torch.bfloat16)


_WO = {"none": K.INT2KV_WO_PLAIN, "plain": K.INT2KV_WO_PLAIN, "folded": K.INT2KV_WO_FOLDED,
       "prepared": K.INT2KV_WO_PREPARED, "prepared_folded": K.INT2KV_WO_PREPARED_FOLDED}


def _attention_inputs(case, seed):
    """Everything of a decode call but the library's own objects."""
    lens, H, Hq, B = _lens(case), case["kv_heads"], case["q_heads"], case["batch"]
    table, pages, phys = _paging(seed, lens)
    g = _gen(seed, 3)
    off = _offsets(seed, H)
    s = dict(lens_host=lens, table_host=table, pages=pages, lens=torch.tensor(lens, dtype=torch.int32, device="cuda"),
             table=table.cuda(), q=_bf16(_randn(g, B, Hq, D)), R_k=_rotations(2 * seed + 1, H),
             R_v=_rotations(2 * seed + 2, H), mu=off, W=_weights(seed, case["d_model"], Hq) if case["d_model"] else None)
    if case["kind"] == "step":
        s["k"], s["v"] = _bf16(_randn(g, B, H, D) + off), _bf16(_randn(g, B, H, D))
        last = torch.tensor(lens) - 1
        s["slots"] = (table[torch.arange(B), last // PAGE] * PAGE + last % PAGE).to(torch.int32).cuda()
    if case["kind"] == "window":
        cap = case["sink"] + case["recent"]
        s["win_k"], s["win_v"] = _bf16(_randn(g, B * cap, H, D)), _bf16(_randn(g, B * cap, H, D))
        s["win_lens"] = torch.full((B,), cap, dtype=torch.int32, device="cuda")
        s["cap"] = cap
    if case["kind"] == "outerr":
        rows = B * case["ctx_hi"]
        s["k_rows"], s["v_rows"] = _bf16(_randn(g, rows, H, D) + off), _bf16(_randn(g, rows, H, D))
        s["pool"] = torch.zeros((len(phys), H, K.RECORD_BYTES_BY_GROUP[case["group"]]), dtype=torch.uint8, device="cuda")
        for b, n in enumerate(pages):  # the cache of those rows: rotated in 64 bits, rounded to 32, quantized
            at = torch.arange(n * PAGE, device="cuda").clamp(max=lens[b] - 1) + b * case["ctx_hi"]
            rot = lambda x, R: torch.matmul(x.double().transpose(0, 1), R.double()).transpose(0, 1).float()  # noqa: E731
            k = rot(s["k_rows"][at].double() - off.double(), s["R_k"]).reshape(n, PAGE, H, D)
            v = rot(s["v_rows"][at], s["R_v"]).reshape(n, PAGE, H, D)
            s["pool"][table[b, :n].long().cuda()] = _records(k, v, case["group"])
    else:
        s["pool"] = _random_pool(seed, phys, H, case["group"])
    return s


def _append_inputs(case, seed):
    n, H = case["tokens"], case["kv_heads"]
    g, off = _gen(seed, 4), _offsets(seed, H)
    blocks = (n + PAGE - 1) // PAGE
    perm = torch.randperm(blocks, generator=torch.Generator().manual_seed(int(seed)))
    t = torch.arange(n)
    s = dict(k=_bf16(_randn(g, n, H, D) + (0 if case["rope"] else off)), v=_bf16(_randn(g, n, H, D)), blocks=blocks,
             slots=(perm[t // PAGE] * PAGE + t % PAGE).to(torch.int32).cuda(), mu=0.1 * off if case["rope"] else off,
             R_k=None, R_v=None, pos=None, cs=None)
    if case["hadamard"]:
        s["R_k"] = K.hadamard_rotation(H)
        s["R_v"] = s["R_k"]
    else:
        s["R_k"], s["R_v"] = _rotations(2 * seed + 1, H), _rotations(2 * seed + 2, H)
    if case["rope"]:
        inv = THETA ** (-torch.arange(0, D, 2, dtype=torch.float64) / D)
        ang = torch.arange(n, dtype=torch.float64)[:, None] * inv
        s["cs"] = torch.cat([ang.cos(), ang.sin()], 1).float().cuda()
        s["pos"] = t.to(torch.int32).cuda()
    return s


def _trace_lens(case, part):
    r = random.Random("%s %d %d %d" % (part, case[part + "_seqs"], case[part + "_lo"], case[part + "_hi"]))
    return [r.randint(case[part + "_lo"], case[part + "_hi"]) for _ in range(case[part + "_seqs"])]


def _calibration_inputs(case, seed):
    H, Hq = case["kv_heads"], case["q_heads"]
    off, s = _offsets(seed, H), {}
    for i, part in enumerate(("calib", "held")):
        g = _gen(seed, 5 + i)
        starts = np.concatenate([[0], np.cumsum(_trace_lens(case, part))]).astype(np.int32)
        T = int(starts[-1])
        s[part] = (_bf16(_randn(g, T, H, D) + off), _bf16(_randn(g, T, H, D)), _bf16(_randn(g, T, Hq, D)), starts)
    s.update(R_k=_rotations(2 * seed + 1, H), R_v=_rotations(2 * seed + 2, H), mu=off,
             W=_weights(seed, case["d_model"], Hq))
    return s


def prepare(case, seed):
    kind = case["kind"]
    if kind == "calibrate":
        s = _calibration_inputs(case, seed)
        s["cfg"] = K.optr_config(case["kv_heads"], case["q_heads"], case["d_model"], group_size=case["group"],
                                 sink=case["sink"], recent=case["recent"], steps=case["steps"],
                                 eval_every=case["eval_every"])
        s["calib"], s["held"] = K.OptrTraces(*s["calib"]), K.OptrTraces(*s["held"])
        n = K.int2kv_optr_workspace_bytes(s["cfg"], s["calib"], s["held"])
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    elif kind == "append":
        s = _append_inputs(case, seed)
        s["cache"] = K.Int2KVCache(s["blocks"], case["kv_heads"], group_size=case["group"])
        s["k_out"] = torch.empty_like(s["k"]) if case["rope"] else None
        s["mu_rk"] = K.int2kv_prepare_mu_rot(s["R_k"], s["mu"])
        s["flags"] = K.INT2KV_HADAMARD_K | K.INT2KV_HADAMARD_V if case["hadamard"] else 0
    else:
        s = _attention_inputs(case, seed)
        H, Hq, B, dm, hi = case["kv_heads"], case["q_heads"], case["batch"], case["d_model"], case["ctx_hi"]
        s["cache"] = K.Int2KVCache(s["pool"].shape[0], H, pool=s["pool"], group_size=case["group"])
        if kind == "outerr":
            n = K.int2kv_output_error_workspace_bytes(B, Hq, H, hi, dm)
            s["out"] = torch.empty((B, Hq, 4), dtype=torch.float32, device="cuda")
        else:
            n = K.int2kv_decode_workspace_bytes(B, Hq, H, hi, dm)
            s["out"] = torch.empty((B, dm) if dm else (B, Hq, D), dtype=torch.float32, device="cuda")
            wo = case["wo"]
            s["wo_format"] = _WO[wo]
            s["W_o"] = s["W"]
            if wo == "folded":
                s["W_o"] = K.int2kv_fold_wo(s["W"], s["R_v"], Hq)
            elif wo.startswith("prepared"):
                s["W_o"] = K.int2kv_prepare_wo(s["W"], s["R_v"] if wo == "prepared_folded" else None, Hq, H)
            if kind == "step":
                s["mu_rk"] = K.int2kv_prepare_mu_rot(s["R_k"], s["mu"])
        s["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    s["case"] = case
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        out = K.int2kv_append_decode(s["cache"], s["k"], s["v"], s["slots"], s["mu_rk"], s["q"], s["table"], s["lens"],
                                     case["ctx_hi"], s["R_k"], s["R_v"], s["W_o"], s["wo_format"], case["d_model"],
                                     out=s["out"], workspace=s["ws"])
        return {"out": out, "pool": s["pool"]}
    if kind == "decode":
        return {"out": K.int2kv_decode(s["cache"], s["q"], s["table"], s["lens"], case["ctx_hi"], s["R_k"], s["R_v"],
                                       s["W_o"], out=s["out"], workspace=s["ws"], wo_format=s["wo_format"],
                                       d_model=case["d_model"])}
    if kind == "window":
        return {"out": K.int2kv_decode_window(s["cache"], s["q"], s["table"], s["lens"], case["ctx_hi"], s["R_k"],
                                              s["R_v"], s["win_k"], s["win_v"], s["win_lens"], s["cap"], s["W_o"],
                                              s["wo_format"], case["d_model"], out=s["out"], workspace=s["ws"])}
    if kind == "append":
        if case["rope"] or case["hadamard"]:
            had = case["hadamard"]
            K.int2kv_quantize_append_rope(s["cache"], s["k"], s["v"], s["slots"], s["pos"], s["cs"],
                                          None if had else s["R_k"], None if had else s["R_v"], s["mu_rk"],
                                          case["clip_k"], case["clip_v"], s["flags"], s["k_out"])
            return {"pool": s["cache"].pool, "k_rope": s["k_out"]}
        K.int2kv_quantize_append(s["cache"], s["k"], s["v"], s["slots"], s["R_k"], s["R_v"], s["mu_rk"],
                                 case["clip_k"], case["clip_v"])
        return {"pool": s["cache"].pool}
    if kind == "outerr":
        got = K.int2kv_output_error(s["cache"], s["q"], s["table"], s["lens"], case["ctx_hi"], s["R_k"], s["R_v"],
                                    s["k_rows"], s["v_rows"], case["ctx_hi"], s["W"], want_dy=case["dy"],
                                    workspace=s["ws"], stats=s["out"])
        return {"stats": got[0], "dy": got[1]} if case["dy"] else {"stats": got}
    return K.int2kv_optr_calibrate(s["cfg"], s["calib"], s["held"], s["R_k"], s["R_v"], s["mu"], s["W"],
                                   workspace=s["ws"])


# ---------------------------------------------------------------------------------------------
# What a pass cannot do without

def work(case):
    H, kind = case["kv_heads"], case["kind"]
    rot = 4 * D * D  # bytes of one rotation matrix
    if kind == "append":
        n, rec = case["tokens"], K.RECORD_BYTES_BY_GROUP[case["group"]] // PAGE
        return {"bytes": n * H * (4 * D + rec + (2 * D if case["rope"] else 0)) + (0 if case["hadamard"] else 2 * H * rot)
                + n * 4 + (n * 4 * (D + 1) if case["rope"] else 0), "flops": 2 * 2 * D * D * n * H}
    if kind == "calibrate":
        Hq, n_last = case["q_heads"], 64
        calib, held = _trace_lens(case, "calib"), _trace_lens(case, "held")
        pairs = lambda ls: sum(min(n_last, L) * L for L in ls) * Hq  # noqa: E731
        evals = 2 + 2 * (case["steps"] // case["eval_every"])
        # per objective: logits and probabilities x values; its gradient takes twice that; plus the row rotations
        fwd = lambda ls: 2 * 2 * D * pairs(ls) + 2 * 2 * D * D * sum(ls) * H  # noqa: E731
        flops = 2 * case["steps"] * 3 * fwd(calib) + evals * fwd(held)
        toks = (sum(calib) + sum(held)) * (2 * H + Hq) * D * 2
        return {"bytes": toks + 2 * case["d_model"] * Hq * D + H * (4 * rot + 2 * 2 * rot), "flops": flops}
    lens, B, Hq, dm = _lens(case), case["batch"], case["q_heads"], case["d_model"]
    rec = K.RECORD_BYTES_BY_GROUP[case["group"]]
    pages = sum((n + PAGE - 1) // PAGE for n in lens)
    nbytes = sum(lens) * H * rec // PAGE + 4 * pages + 4 * B + B * Hq * D * 2 + 2 * H * rot
    flops = 4 * D * Hq * sum(lens) + 2 * 2 * D * D * B * Hq
    if kind == "outerr":
        nbytes += sum(lens) * H * D * 4 + 2 * dm * Hq * D + B * Hq * 16 + (B * Hq * 8 * dm if case["dy"] else 0)
        return {"bytes": nbytes, "flops": 10 * D * Hq * sum(lens) + 2 * 2 * D * dm * B * Hq}
    if kind == "window":
        cap = case["sink"] + case["recent"]
        nbytes += B * cap * H * D * 4
        flops += 4 * D * Hq * B * cap
    if kind == "step":
        nbytes += B * H * (4 * D + rec // PAGE)
    nbytes += 2 * dm * Hq * D + 4 * B * dm if dm else 4 * B * Hq * D
    return {"bytes": nbytes, "flops": flops + 2 * B * dm * Hq * D}


def tolerance(case):
    return {
        # fp16 query operands, probabilities and (prepared) weights; cache bytes move only at rounding ties
        "step": {"rel": 5e-3, "max": 5e-2, "differ": 1e-4},
        "decode": {"rel": 5e-3, "max": 5e-2},
        "window": {"rel": 5e-3, "max": 5e-2},
        # bytes move only where the fp32 rotation's last bits cross a rounding boundary of a code or an fp16 scale or zero
        # (3e-5 of the bytes between the write and a correctly rounded rotation); post-RoPE keys are rounded once
        "append": {"rel": 1e-4, "max": 1e-2, "differ": 1.5e-4},
        # fp32 sums throughout
        "outerr": {"rel": 1e-5, "max": 1e-3},
        # fp64 throughout (1e-12 seen), rotations rounded to fp32; a code that flips at a tie moves a step by about 1e-6
        "calibrate": {"rel": 1e-6, "max": 1e-4},
    }[case["kind"]]


# ---------------------------------------------------------------------------------------------
# The same outputs in 64 bits, in plain torch

def _heads_of(q, H):
    """Queries [Hq, 128] by KV head: fp64 [H, gq, 128]."""
    return q.double().reshape(H, -1, D)


def _exact_attention(case, seed):
    s = _attention_inputs(case, seed)
    H, Hq, B, group = case["kv_heads"], case["q_heads"], case["batch"], case["group"]
    Rk, Rv = s["R_k"].double(), s["R_v"].double()
    o = torch.zeros((B, Hq, D), dtype=torch.float64, device="cuda")
    do = torch.zeros((B, Hq, 2, D), dtype=torch.float64, device="cuda")
    if case["kind"] == "step":
        kr = (torch.matmul(s["k"].double().transpose(0, 1), Rk) - torch.matmul(s["mu"].double()[:, None], Rk)).float()
        vr = torch.matmul(s["v"].double().transpose(0, 1), Rv).float()
        new_k, new_v = (_dequantize(*_quantize(x.transpose(0, 1), group), group) for x in (kr, vr))
    for b, n in enumerate(s["lens_host"]):
        k, v = _rows_of(s["pool"][s["table_host"][b, :s["pages"][b]].long().cuda()], group)
        k, v = k.reshape(-1, H, D)[:n].clone(), v.reshape(-1, H, D)[:n].clone()
        if case["kind"] == "step":
            k[n - 1], v[n - 1] = new_k[b], new_v[b]
        q = _heads_of(s["q"][b], H)
        k, v = k.transpose(0, 1), torch.matmul(v.transpose(0, 1), Rv.transpose(1, 2))
        a = torch.matmul(torch.matmul(q, Rk), k.transpose(1, 2)) * SCALE
        if case["kind"] == "window":
            rows = slice(b * s["cap"], (b + 1) * s["cap"])
            wk, wv = (s[x][rows].double().transpose(0, 1) for x in ("win_k", "win_v"))
            a, v = torch.cat([a, torch.matmul(q, wk.transpose(1, 2)) * SCALE], -1), torch.cat([v, wv], 1)
        p = torch.softmax(a, -1)
        ob = torch.matmul(p, v)
        o[b] = ob.reshape(Hq, D)
        if case["kind"] == "outerr":
            rows = slice(b * case["ctx_hi"], b * case["ctx_hi"] + n)
            kf, vf = (s[x][rows].double().transpose(0, 1) for x in ("k_rows", "v_rows"))
            pf = torch.softmax(torch.matmul(q, (kf - s["mu"].double()[:, None]).transpose(1, 2)) * SCALE, -1)
            mid = torch.matmul(p, vf)
            do[b] = torch.stack([mid - torch.matmul(pf, vf), ob - mid], 2).reshape(Hq, 2, D)
    if case["kind"] == "outerr":
        W = s["W"].double().reshape(-1, Hq, D)
        dy = torch.stack([torch.matmul(do[:, j], W[:, j].t().contiguous()) for j in range(Hq)], 1)
        ek, ev = dy[:, :, 0], dy[:, :, 1]
        stats = torch.stack([((ek + ev) ** 2).sum(-1), (ek ** 2).sum(-1), (ev ** 2).sum(-1), (ek * ev).sum(-1)], -1)
        return {"stats": stats, "dy": dy} if case["dy"] else {"stats": stats}
    out = torch.matmul(o.reshape(B, -1), s["W"].double().t().contiguous()) if case["d_model"] else o
    return {"out": out, "pool": None} if case["kind"] == "step" else {"out": out}


def _exact_append(case, seed):
    s = _append_inputs(case, seed)
    if not case["rope"]:
        return None  # packed bytes only
    x, half = s["k"].double(), D // 2
    c, sn = s["cs"][:, None, :half].double(), s["cs"][:, None, half:].double()
    lo, hi = x[..., :half], x[..., half:]
    return {"pool": None, "k_rope": torch.cat([lo * c - hi * sn, hi * c + lo * sn], -1)}


class _Rounded(torch.autograd.Function):
    """The cache's quantizer on the fp32 rounding of fp64 rows, with the straight-through gradient: it passes where an
    element lies inside its group's clipped range."""

    @staticmethod
    def forward(ctx, z, clip, group):
        z32 = z.float()
        g = z32.reshape(z.shape[:-1] + (D // group, group))
        c = torch.tensor(clip, dtype=torch.float32, device=z.device)
        lo, hi = c * g.amin(-1, keepdim=True), c * g.amax(-1, keepdim=True)
        ctx.save_for_backward(((g >= lo) & (g <= hi)).reshape(z.shape))
        return _dequantize(*_quantize(z32, group, clip), group)

    @staticmethod
    def backward(ctx, grad):
        return grad * ctx.saved_tensors[0], None, None


def _exact_calibration(case, seed):
    s = _calibration_inputs(case, seed)
    H, Hq, dm, group = case["kv_heads"], case["q_heads"], case["d_model"], case["group"]
    gq, n_last, clip = Hq // H, 64, (0.96, 0.92)
    W = s["W"].double().reshape(dm, Hq, D)
    gram = torch.stack([torch.matmul(W[:, j].t().contiguous(), W[:, j]) for j in range(Hq)]).reshape(H, gq, D, D)

    def split(part):
        k, v, q, starts = s[part]
        seqs = []
        for a, e in zip(starts[:-1].tolist(), starts[1:].tolist()):
            L = e - a
            t = torch.arange(max(0, L - n_last), L, device="cuda")
            u = torch.arange(L, device="cuda")
            causal = u[None] <= t[:, None]
            int2 = causal & (u[None] >= case["sink"]) & (u[None] <= t[:, None] - case["recent"])
            qs = q[a:e].double()[t].reshape(len(t), H, gq, D).permute(1, 2, 0, 3).reshape(H, -1, D)
            seqs.append(dict(k=k[a:e].double().transpose(0, 1) - s["mu"].double()[:, None], q=qs,
                             v=v[a:e].double().transpose(0, 1).contiguous(), rows=len(t),
                             causal=causal.repeat(gq, 1), int2=int2.repeat(gq, 1)))
        return seqs

    def rotation(A, R0):
        return torch.matmul(R0.double(), torch.linalg.matrix_exp(A - A.transpose(1, 2)))

    def logits(d, A):
        R = rotation(A, s["R_k"])
        eff = torch.matmul(_Rounded.apply(torch.matmul(d["k"], R), clip[0], group), R.transpose(1, 2))
        full = torch.matmul(d["q"], d["k"].transpose(1, 2)) * SCALE
        quant = torch.matmul(d["q"], eff.transpose(1, 2)) * SCALE
        mask = lambda x: x.masked_fill(~d["causal"], -1.0e300)  # noqa: E731
        return mask(full), mask(torch.where(d["int2"], quant, full))

    def projected(e, d):
        e = e.reshape(H, gq, d["rows"], D)
        return (torch.matmul(e, gram) * e).sum((1, 2, 3)) / dm

    def key_loss(A, seqs):
        total = 0.0
        for d in seqs:
            full, mixed = logits(d, A)
            lp, lk = torch.log_softmax(full, -1), torch.log_softmax(mixed, -1)
            p, pk = lp.exp(), lk.exp()
            kl = torch.where(d["causal"], p * (lp - lk), torch.zeros_like(p)).sum((1, 2))
            total = total + kl + projected(torch.matmul(pk - p, d["v"]), d)
        return total / sum(d["rows"] * gq for d in seqs)

    def value_loss(A, seqs):
        R, total = rotation(A, s["R_v"]), 0.0
        for d in seqs:
            eff = torch.matmul(_Rounded.apply(torch.matmul(d["v"], R), clip[1], group), R.transpose(1, 2))
            total = total + projected(torch.matmul(d["p"], eff - d["v"]), d)
        return total / sum(d["rows"] * gq for d in seqs)

    parts, steps, ev = {x: split(x) for x in ("calib", "held")}, case["steps"], case["eval_every"]
    res, hist = [], []
    for loss_of in (key_loss, value_loss):
        A = torch.zeros((H, D, D), dtype=torch.float64, device="cuda", requires_grad=True)
        opt = torch.optim.Adam([A], lr=0.02)
        curve, held = [], [loss_of(A.detach(), parts["held"])]
        best, kept = held[0].clone(), A.detach().clone()
        for i in range(1, steps + 1):
            opt.zero_grad()
            loss = loss_of(A, parts["calib"])
            loss.sum().backward()  # the heads are independent
            curve.append(loss.detach())
            opt.step()
            if i % ev == 0:
                held.append(loss_of(A.detach(), parts["held"]))
                better = held[-1] < best
                best = torch.where(better, held[-1], best)
                kept = torch.where(better[:, None, None], A.detach(), kept)
        res.append(kept)
        hist.append(torch.stack(curve + held, 1))
        if loss_of is key_loss:
            for d in parts["calib"] + parts["held"]:
                d["p"] = torch.softmax(logits(d, kept)[1], -1) * d["int2"]
    return {"R_k": rotation(res[0], s["R_k"]), "R_v": rotation(res[1], s["R_v"]), "A_k": res[0], "A_v": res[1],
            "history": torch.stack(hist)}


def exact(case, seed):
    with torch.no_grad() if case["kind"] != "calibrate" else torch.enable_grad():
        if case["kind"] == "calibrate":
            return {k: v.detach() for k, v in _exact_calibration(case, seed).items()}
        return _exact_append(case, seed) if case["kind"] == "append" else _exact_attention(case, seed)
