"""The work that programs have this library do, as cases that can be timed and compared.

Six kinds, each through the binding's public calls:

  step     sali_step frame by frame on one stream: a caller that gets one frame at a time
  clip     a stretch of video through the batched calls: analysis a batch ahead on image streams, storage
           (and read-back) on another, as the benchmark and a serving loop chain them
  flow     sali_flow_score of a frame pair: the temporal filter as a call of its own, with the dense flow
  saliency sali_saliency_pool of a frame: the spatial filter as a call of its own, with the map
  kv       sali_kv_compress of frames whose scores come from elsewhere, then sali_kv_decompress
  attend   one decode (or prompt) step: attention of every layer over the cached frames

Sizes are those of the repository's workloads (336x336, 640x360, 1920x1080; 7B- and 13B-shaped K/V; 8 K/V heads
with grouped queries; the 784-patch budget) and ranges around them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_14236_amd import binding

DEV = "cuda:0"
TOKENS, HEAD_DIM, GROUP = 576, 128, 32
ROW_BYTES = (256.0, 144.0, 88.0)            # a pool row: fp16; int8 codes + scales; int4 codes + scales + zeros


# ------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # One layer of a grouped-query model (8 K/V heads): the smallest call a caller makes, all launch latency.
        dict(name="kv-1layer-8h", kind="kv", frames=1, layers=1, heads=8, mode=1, k16=173, k8=403, k4=0),
        # A live caller: one frame at a time on one stream, one layer of 32 heads, threshold tiers, a duplicate frame.
        dict(name="step-336-1layer", kind="step", h=336, w=336, levels=3, frames=8, batch=1, motion="mixed", layers=1,
             heads=32, mode=0, k16=0, k8=0, k4=0, readback=False),
        # The headline: 7B-shaped K/V, int8 background, four frames per call, read back while the next are analysed.
        dict(name="clip-336-7b", kind="clip", h=336, w=336, levels=3, frames=8, batch=4, motion="moving", layers=32,
             heads=32, mode=1, k16=173, k8=403, k4=0, readback=True),
        # A 30 fps stream with near-static runs, four layers of the 7B shape, sixteen frames per call, no read-back.
        dict(name="clip-640x360-4layer", kind="clip", h=360, w=640, levels=3, frames=32, batch=16, motion="mixed",
             layers=4, heads=32, mode=1, k16=249, k8=56, k4=168, readback=False),
        # Flow-heavy: full HD, five pyramid levels, sub-pixel motion up to 12 px, 13B-shaped K/V, int4 background.
        dict(name="clip-1080p-13b", kind="clip", h=1080, w=1920, levels=5, frames=4, batch=4, motion="subpixel",
             layers=40, heads=40, mode=1, k16=173, k8=0, k4=403, readback=False),
        # A frame size nobody tuned for (neither even nor a multiple of a tile), threshold tiers, few heads.
        dict(name="clip-241x427-odd", kind="clip", h=241, w=427, levels=4, frames=6, batch=3, motion="moving", layers=2,
             heads=5, mode=0, k16=0, k8=0, k4=0, readback=True),
        # The temporal filter of one pair at the model's own input size.
        dict(name="flow-336", kind="flow", h=336, w=336, levels=3, motion="moving"),
        # The same at full HD: the largest single image a caller passes.
        dict(name="flow-1080p", kind="flow", h=1080, w=1920, levels=5, motion="subpixel"),
        # The spatial filter alone with its map, at the stream's source size.
        dict(name="saliency-640x360", kind="saliency", h=360, w=640, motion="moving"),
        # Decode steps of a long cached video: one query per head, eight layers, each layer's rows read once.
        dict(name="attend-1q-32h", kind="attend", frames=20, layers=8, heads=32, q_per_kv=1, mode=1, k16=173, k8=403, k4=0),
        # The paper's own setting: 32 query heads over 8 K/V heads, a small cache (budget of 784 patches), all layers.
        dict(name="attend-4q-8h-small", kind="attend", frames=2, layers=32, heads=8, q_per_kv=4, mode=1, k16=124, k8=28,
             k4=84),
        # A prompt of 32 tokens against the cached video: the matrix-core path.
        dict(name="attend-32q-32h", kind="attend", frames=20, layers=4, heads=32, q_per_kv=32, mode=1, k16=173, k8=200,
             k4=203),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_counts(rng):
    """Tokens per tier (fp16, int8, int4), the rest pruned."""
    kept = rng.choice((TOKENS, TOKENS, rng.randint(200, TOKENS)))
    k16 = int(kept * rng.uniform(0.0, 0.6))
    rest = kept - k16
    k8 = rng.choice((0, rest, rng.randint(0, rest)))
    return k16, k8, rest - k8


def _draw_size(rng):
    """A frame of any shape between thumbnail and full HD, odd sizes included; levels the smallest side allows."""
    h = _log_int(rng, 97, 1080)
    w = min(1920, max(97, int(h * rng.uniform(0.6, 1.78))))
    return h, w, rng.randint(2, 5 if min(h, w) >= 200 else 3)


def draw(rng):
    kind = rng.choice(("step", "clip", "clip", "flow", "flow", "saliency", "kv", "attend", "attend", "attend"))
    k16, k8, k4 = _draw_counts(rng)
    mode = rng.choice((0, 1, 1))
    if kind in ("flow", "saliency"):
        h, w, levels = _draw_size(rng)
        case = dict(kind=kind, h=h, w=w, motion=rng.choice(("moving", "subpixel")))
        if kind == "flow":
            case["levels"] = levels
        return case
    heads = rng.choice((4, 5, 8, 16, 32, 40))
    if kind in ("step", "clip"):
        h, w, levels = _draw_size(rng)
        layers = _log_int(rng, 1, 32)
        batch = 1 if kind == "step" else rng.choice((2, 3, 4, 8, 16))
        # no more K/V than the largest listed clip moves, no more pixels than four full HD frames
        most = min(40, int(1.8e9 / (layers * 2 * heads * TOKENS * HEAD_DIM * 2)), int(4 * 1080 * 1920 / (h * w)))
        frames = max(2, min(most, rng.randint(2, 2 * batch + 6)))
        return dict(kind=kind, h=h, w=w, levels=levels, frames=frames, batch=batch,
                    motion=rng.choice(("moving", "mixed", "subpixel")), layers=layers, heads=heads, mode=mode,
                    k16=k16, k8=k8, k4=k4, readback=rng.random() < 0.5)
    if kind == "kv":
        layers = _log_int(rng, 1, 32)
        frames = max(1, min(4, int(1.2e9 / (layers * 2 * heads * TOKENS * HEAD_DIM * 2))))
        return dict(kind=kind, frames=frames, layers=layers, heads=heads, mode=mode, k16=k16, k8=k8, k4=k4)
    q_per_kv = rng.choice((1, 2, 4, 8, rng.randint(9, 64), 32))
    return dict(kind="attend", frames=_log_int(rng, 1, 24), layers=rng.randint(1, 4), heads=heads, q_per_kv=q_per_kv,
                mode=mode, k16=k16, k8=k8, k4=k4)


# ------------------------------------------------------------------------------------------ inputs
def _generator(seed, *salt):
    g = torch.Generator(device=DEV)
    mix = 0x9E3779B97F4A7C15
    x = seed & 0xFFFFFFFF
    for s in salt:
        x = ((x ^ (s + 1)) * mix + 0x1234567) & 0x7FFFFFFFFFFFFFFF
    g.manual_seed(x)
    return g


def _uniform(g, n, lo, hi):
    return (lo + (hi - lo) * torch.rand(n, generator=g, device=DEV)).tolist()


def _frames(case, seed, n):
    """n RGB uint8 frames [h, w, 3]: low-frequency sinusoid background, six textured ellipses that move (whole pixels,
    or sub-pixel at up to 12 px per 1080 rows), fresh sensor noise of two grey levels; "mixed" motion holds still or
    repeats the frame before in places."""
    h, w, motion = case["h"], case["w"], case["motion"]
    g = _generator(seed, 1)
    yy = torch.arange(h, device=DEV, dtype=torch.float32)[:, None]
    xx = torch.arange(w, device=DEV, dtype=torch.float32)[None, :]
    tau = 2.0 * math.pi
    lam_x, lam_y = _uniform(g, 3, 0.5 * w, 1.5 * w), _uniform(g, 3, 0.5 * w, 1.5 * w)
    ph_x, ph_y = _uniform(g, 3, 0.0, tau), _uniform(g, 3, 0.0, tau)
    background = torch.stack([128.0 + 40.0 * torch.sin(tau * xx / lam_x[c] + ph_x[c]) * torch.sin(tau * yy / lam_y[c] + ph_y[c])
                              for c in range(3)], dim=2)
    tex = h / 336.0 if motion == "subpixel" else 1.0
    ellipses = []
    for _ in range(6):
        ax, ay = _uniform(g, 2, w / 16.0, w / 6.0)
        cx, cy, ang = _uniform(g, 1, 0.0, w)[0], _uniform(g, 1, 0.0, h)[0], _uniform(g, 1, 0.0, math.pi)[0]
        col = _uniform(g, 3, 40.0, 215.0)
        l1, l2 = (v * max(1.0, tex) for v in _uniform(g, 2, 6.0, 12.0))
        if motion == "subpixel":
            mag, th = _uniform(g, 1, 2.0, 12.0)[0] * min(1.0, h / 1080.0 + 0.2), _uniform(g, 1, 0.0, tau)[0]
            vx, vy = mag * math.cos(th), mag * math.sin(th)
        else:
            vx, vy = (round(v) for v in _uniform(g, 2, -4.4, 4.4))
            if vx == 0 and vy == 0:
                vx = 2
        ellipses.append((ax, ay, cx, cy, ang, col, l1, l2, float(vx), float(vy)))
    out, moved = [], 0
    for t in range(n):
        hold = motion == "mixed" and t % 8 in (3, 5, 6)
        if hold and t % 8 == 3:
            out.append(out[-1].clone())                     # a byte copy of the frame before
            continue
        if t > 0 and not hold:
            moved += 1
        img = background.clone()
        for ax, ay, cx, cy, ang, col, l1, l2, vx, vy in ellipses:
            dx = torch.remainder(xx - (cx + vx * moved) + w / 2.0, w) - w / 2.0
            dy = torch.remainder(yy - (cy + vy * moved) + h / 2.0, h) - h / 2.0
            p = math.cos(ang) * dx + math.sin(ang) * dy
            q = -math.sin(ang) * dx + math.cos(ang) * dy
            inside = ((p / ax) ** 2 + (q / ay) ** 2 <= 1.0)[:, :, None]
            wave = (30.0 * torch.sin(tau * p / l1) * torch.sin(tau * q / l2))[:, :, None]
            img = torch.where(inside, torch.tensor(col, device=DEV) + wave, img)
        img = img + 2.0 * torch.randn(img.shape, generator=g, device=DEV)
        out.append(img.round_().clamp_(0, 255).to(torch.uint8).contiguous())
    return out


def _kv(case, seed, t):
    """K/V of frame t, fp16 [layers, 2, heads, 576, 128]: N(0, 1) times a per-channel lognormal(0, 0.5) scale."""
    layers, heads = case["layers"], case["heads"]
    gs = _generator(seed, 2)
    scale = torch.exp(0.5 * torch.randn((layers, 2, heads, 1, HEAD_DIM), generator=gs, device=DEV))
    g = _generator(seed, 3, t)
    out = torch.empty((layers, 2, heads, TOKENS, HEAD_DIM), dtype=torch.float16, device=DEV)
    for layer in range(layers):
        z = torch.randn(out.shape[1:], generator=g, device=DEV)
        out[layer] = (z * scale[layer]).to(torch.float16)
    return out


def _scores(seed, t):
    """576 saliency scores as the spatial filter gives them for 14x14 patches: floor(q * 2^15 / 196) / 2^16 with many
    low ones, ties and zeros among them."""
    g = _generator(seed, 4, t)
    u = torch.rand(TOKENS, generator=g, device=DEV)
    q = torch.clamp((u ** 2.5 * 420.0) - 12.0, 0.0, 392.0).to(torch.int64)
    return ((q * 32768) // 196).to(torch.float32) / 65536.0


def _queries(case, seed):
    g = _generator(seed, 5)
    shape = (case["layers"], case["heads"] * case["q_per_kv"], HEAD_DIM)
    return torch.randn(shape, generator=g, device=DEV).to(torch.float16)


# ------------------------------------------------------------------------------------------ prepare
def _context(case, frames, h=336, w=336, levels=3):
    cap = [max(1, (k if case["mode"] == 1 else TOKENS) * frames) for k in (case["k16"], case["k8"], case["k4"])]
    cfg = binding.make_config(h, w, flow_levels=levels, tier_mode=case["mode"], k_fp16=case["k16"], k_int8=case["k8"],
                              k_int4=case["k4"], n_layers=case["layers"], n_heads=case["heads"], cap_fp16=cap[0],
                              cap_int8=cap[1], cap_int4=cap[2], max_frames=frames)
    ctx = binding.SaliContext(cfg, DEV)
    ctx.pools.zero_()                                   # rows nobody writes are outputs too: give them a value
    return ctx


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("flow", "saliency"):
        h, w = case["h"], case["w"]
        s["ctx"] = binding.SaliContext(binding.make_config(h, w, flow_levels=case.get("levels", 1), n_heads=1), DEV)
        s["rgb"] = _frames(case, seed, 2 if kind == "flow" else 1)
        if kind == "flow":
            s["uv"] = torch.empty((2, h, w), dtype=torch.float32, device=DEV)
            s["motion"] = torch.empty(TOKENS, dtype=torch.float32, device=DEV)
            s["gate"] = torch.empty(4, dtype=torch.int32, device=DEV)
        else:
            s["map"] = torch.empty((h, w), dtype=torch.uint8, device=DEV)
            s["scores"] = torch.empty(TOKENS, dtype=torch.float32, device=DEV)
        return s
    n = case["frames"]
    dense = (case["layers"], 2, case["heads"], TOKENS, HEAD_DIM)
    if kind in ("step", "clip"):
        s["ctx"] = _context(case, n, case["h"], case["w"], case["levels"])
        s["rgb"] = _frames(case, seed, n)
        s["kv"] = [_kv(case, seed, t) for t in range(n)]
        if case["readback"]:
            s["dense"] = [torch.empty(dense, dtype=torch.float16, device=DEV) for _ in range(n)]
            s["valid"] = torch.empty((n, TOKENS), dtype=torch.uint8, device=DEV)
        if kind == "clip":
            s["image_streams"] = [torch.cuda.Stream() for _ in range(2)]
            s["kv_stream"] = torch.cuda.Stream()
        return s
    s["ctx"] = ctx = _context(case, n)
    if kind == "kv":
        s["kv"] = [_kv(case, seed, t) for t in range(n)]
        s["scores"] = [_scores(seed, t) for t in range(n)]
        s["dense"] = [torch.empty(dense, dtype=torch.float16, device=DEV) for _ in range(n)]
        s["valid"] = torch.empty((n, TOKENS), dtype=torch.uint8, device=DEV)
        return s
    for t in range(n):                                  # attend: the video is in the cache already
        ctx.kv_compress(_kv(case, seed, t), _scores(seed, t), t)
    s["q"] = _queries(case, seed)
    s["out"] = torch.empty(s["q"].shape, dtype=torch.float32, device=DEV)
    s["lse"] = torch.empty(s["q"].shape[:2], dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------------------------------ run
def _stored(s):
    """The compressed cache as it lies in memory (its layout is part of the C ABI), and what was read back."""
    out = dict(s["ctx"].pool_views_flat())
    if "dense" in s:
        out["dense"] = s["dense"]
        out["valid"] = s["valid"]
    return out


def _run_clip(s):
    case, ctx = s["case"], s["ctx"]
    n, batch = case["frames"], case["batch"]
    here, images, kvs = torch.cuda.current_stream(), s["image_streams"], s["kv_stream"]
    ctx.reset()
    for st in images + [kvs]:
        st.wait_stream(here)
    calls = [range(t, min(n, t + batch)) for t in range(0, n, batch)]

    def analyse(b):
        if b < len(calls):
            ctx.analyze_batch([s["rgb"][t] for t in calls[b]], calls[b][0], images[b % len(images)])

    analyse(0)
    for b, frames in enumerate(calls):
        analyse(b + 1)
        ctx.store_batch([s["kv"][t] for t in frames], frames[0], kvs)
        if case["readback"]:
            ctx.kv_decompress_batch(frames[0], [s["dense"][t] for t in frames], s["valid"][frames[0]:], kvs)
    for st in images + [kvs]:
        here.wait_stream(st)
    return _stored(s)


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "flow":
        ctx.flow_score(s["rgb"][0], s["rgb"][1], s["uv"], s["motion"], s["gate"])
        return {"uv": s["uv"], "motion": s["motion"], "static_and_redundant": s["gate"][0:3:2]}
    if kind == "saliency":
        ctx.saliency_pool(s["rgb"][0], s["map"], s["scores"])
        return {"map": s["map"], "scores": s["scores"]}
    if kind == "clip":
        return _run_clip(s)
    if kind == "step":
        ctx.reset()
        for t in range(case["frames"]):
            ctx.step(s["rgb"][t], s["kv"][t], t)
            if case["readback"]:
                ctx.kv_decompress(t, s["dense"][t], s["valid"][t])
        return _stored(s)
    if kind == "kv":
        ctx.reset()
        for t in range(case["frames"]):
            ctx.kv_compress(s["kv"][t], s["scores"][t], t)
        for t in range(case["frames"]):
            ctx.kv_decompress(t, s["dense"][t], s["valid"][t])
        return _stored(s)
    scale = 1.0 / math.sqrt(HEAD_DIM)
    for layer in range(case["layers"]):
        if case["q_per_kv"] == 1:
            ctx.attend_decode(layer, s["q"][layer], 0, case["frames"], scale, s["out"][layer], s["lse"][layer])
        else:
            ctx.attend_decode_gqa(layer, s["q"][layer], case["q_per_kv"], 0, case["frames"], scale, s["out"][layer],
                                  s["lse"][layer])
    return {"out": s["out"], "lse": s["lse"]}


# ------------------------------------------------------------------------------------------ work, tolerance
def work(case):
    """What a pass cannot do without.  Threshold tiers depend on the content: counted as 150 fp16, 60 int8, 100 int4
    tokens a frame."""
    kind = case["kind"]
    if kind in ("flow", "saliency"):
        px = case["h"] * case["w"]
        # flow: per pixel of the pyramid (4/3 of the frame) an expansion and three updates: terms, two window
        # passes of 5 x 11 multiply-adds, the solve
        if kind == "flow":
            return {"bytes": 2 * 3 * px + 8 * px + 4 * TOKENS, "flops": px * 4 / 3 * (2 * 70 + 3 * (2 * 110 + 90))}
        return {"bytes": 3 * px + px + 4 * TOKENS, "flops": px * 250}
    kept = (case["k16"], case["k8"], case["k4"]) if case["mode"] == 1 else (150, 60, 100)
    frames, rows = case["frames"], case["layers"] * 2 * case["heads"]
    packed = sum(k * b for k, b in zip(kept, ROW_BYTES))
    if kind == "attend":
        q = case["layers"] * case["heads"] * case["q_per_kv"]
        return {"bytes": frames * rows * packed + q * (2 + 4) * HEAD_DIM + 4 * q, "flops": 4 * HEAD_DIM * q * frames * sum(kept)}
    stored = frames
    if kind in ("step", "clip") and case["motion"] == "mixed":
        stored = sum(1 for t in range(frames) if t % 8 not in (3, 5, 6))
    nbytes = stored * rows * (sum(kept) * 256.0 + packed)
    if kind == "kv" or case["readback"]:
        nbytes += frames * rows * (packed + TOKENS * 256.0)
    flops = stored * rows * sum(kept) * HEAD_DIM * 4
    if kind != "kv":
        px = case["h"] * case["w"]
        nbytes += frames * 5 * px
        flops += frames * px * (4 / 3 * (70 + 3 * (2 * 110 + 90)) + 250)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # about four times the largest distance from 64 bits seen over some forty sizes
    if case["kind"] == "flow":
        # fp32 through the pyramid's levels and their updates: 1.4e-6, single vectors 2.6e-5
        return {"rel": 6e-6, "max": 1.2e-4}
    if case["kind"] == "attend":
        if case["q_per_kv"] <= 8:
            return {"rel": 2e-6, "max": 3e-5}           # fp32 sums: 4.6e-7, single values 6.4e-6
        return {"rel": 1.1e-3, "max": 2e-2}             # fp16 operands of the matrix cores: 2.7e-4, 5.3e-3
    return "exact"                                      # codes, scales, tiers and maps are integers or defined bit by bit


# ------------------------------------------------------------------------------------------ exact results
def exact(case, seed):
    if case["kind"] == "flow":
        return _exact_flow(case, seed)
    if case["kind"] == "attend":
        return _exact_attention(case, seed)
    if case["kind"] == "kv":
        return _exact_read_back(case, seed)
    return None


def _tiers(case, scores):
    """Tier of every token: 0 fp16, 1 int8, 2 int4, 3 pruned."""
    tier = torch.full((TOKENS,), 3, device=DEV)
    if case["mode"] == 0:
        for code, tau in ((2, 0.03), (1, 0.15), (0, 0.30)):
            tier[scores > np.float32(tau).item()] = code
        return tier
    order = torch.sort(scores, descending=True, stable=True).indices      # ties: the lower token first
    edges = (0, case["k16"], case["k16"] + case["k8"], case["k16"] + case["k8"] + case["k4"])
    for code in range(3):
        tier[order[edges[code]:edges[code + 1]]] = code
    return tier


def _dequantised(x, tier):
    """The numbers that the stored codes, fp32 scales and fp16 zero-points of rows x [..., tokens, 128] stand for, in
    64 bits; the codes by the definition's fp32 operations."""
    out = torch.zeros(x.shape, dtype=torch.float64, device=DEV)
    out[..., tier == 0, :] = x[..., tier == 0, :].double()
    for code in (1, 2):
        v = x[..., tier == code, :].float()
        if v.shape[-2] == 0:
            continue
        g = v.view(*v.shape[:-1], HEAD_DIM // GROUP, GROUP)
        if code == 1:
            zero = torch.zeros_like(g[..., :1])
            span, steps = g.abs().amax(-1, keepdim=True), 127.0
        else:
            zero = g.amin(-1, keepdim=True)
            span, steps = g.amax(-1, keepdim=True) - zero, 15.0
        k = torch.full_like(span, steps)
        scale = torch.where(span > 0, span / k, torch.zeros_like(span))
        inv = torch.where(span > 0, k / span, torch.zeros_like(span))
        q = torch.round((g - zero) * inv)
        out[..., tier == code, :] = (q.double() * scale.double() + zero.double()).view(v.shape)
    return out


def _exact_read_back(case, seed):
    n = case["frames"]
    if n * case["layers"] * case["heads"] > 512:
        return None                                     # gigabytes of 64-bit numbers
    dense, valid = [], []
    for t in range(n):
        tier = _tiers(case, _scores(seed, t))
        dense.append(_dequantised(_kv(case, seed, t), tier))
        valid.append((tier != 3).to(torch.uint8))
    out = {k: None for k in ("fp16", "codes8", "scale8", "codes4", "scale4", "zero4")}
    out["dense"], out["valid"] = dense, torch.stack(valid)
    return out


def _exact_attention(case, seed):
    n, heads, per = case["frames"], case["heads"], case["q_per_kv"]
    q = _queries(case, seed).double().view(case["layers"], heads, per, HEAD_DIM)
    tiers = [_tiers(case, _scores(seed, t)) for t in range(n)]
    kvs = [_kv(case, seed, t) for t in range(n)]
    outs, lses = [], []
    for layer in range(case["layers"]):
        k, v = [], []
        for t in range(n):
            rows = _dequantised(kvs[t][layer], tiers[t])[:, :, tiers[t] != 3, :]
            k.append(rows[0])
            v.append(rows[1])
        k, v = torch.cat(k, dim=1), torch.cat(v, dim=1)
        s = torch.bmm(q[layer], k.transpose(1, 2).contiguous()) / math.sqrt(HEAD_DIM)
        lses.append(torch.logsumexp(s, dim=-1).reshape(-1))
        outs.append(torch.bmm(torch.softmax(s, dim=-1), v).reshape(-1, HEAD_DIM))
    return {"out": torch.stack(outs), "lse": torch.stack(lses)}


def _clamp_rows(x, offset, axis):
    """x shifted by offset along an axis, the border repeated."""
    n = x.shape[axis]
    i = (torch.arange(n, device=DEV) + offset).clamp_(0, n - 1)
    return x.index_select(axis, i)


def _filter(x, taps, radius):
    """Correlation along both axes with the same taps, the border repeated."""
    for axis in (0, 1):
        x = sum(taps[k + radius] * _clamp_rows(x, k, axis) for k in range(-radius, radius + 1))
    return x


def _gaussian(radius, sigma):
    t = np.exp(-np.arange(-radius, radius + 1, dtype=np.float64) ** 2 / (2.0 * sigma * sigma))
    return t / t.sum()


def _expansion(f):
    """A (xx, xy, yy) and b (x, y) of the 7x7 Gaussian-weighted quadratic fit."""
    g = _gaussian(3, 1.5)
    k = np.arange(-3, 4, dtype=np.float64)
    m2, m4 = float((g * k ** 2).sum()), float((g * k ** 4).sum())

    def moment(py, px):
        y = sum(float(g[i] * k[i] ** py) * _clamp_rows(f, i - 3, 0) for i in range(7))
        return sum(float(g[i] * k[i] ** px) * _clamp_rows(y, i - 3, 1) for i in range(7))

    s0 = moment(0, 0)
    den = m4 - m2 * m2
    return torch.stack([(moment(0, 2) - m2 * s0) / den, moment(1, 1) / (2.0 * m2 * m2), (moment(2, 0) - m2 * s0) / den,
                        moment(0, 1) / m2, moment(1, 0) / m2])


def _bilinear(fields, y, x):
    """fields [c, h, w] at real coordinates, clamped to the image."""
    h, w = fields.shape[1:]
    y, x = y.clamp(0.0, h - 1.0), x.clamp(0.0, w - 1.0)
    y0, x0 = y.floor(), x.floor()
    wy, wx = y - y0, x - x0
    y0, x0 = y0.long(), x0.long()
    y1, x1 = (y0 + 1).clamp(max=h - 1), (x0 + 1).clamp(max=w - 1)
    flat = fields.reshape(fields.shape[0], -1)

    def at(iy, ix):
        return flat[:, (iy * w + ix).reshape(-1)].view(fields.shape[0], *iy.shape)

    return (at(y0, x0) * (1 - wx) + at(y0, x1) * wx) * (1 - wy) + (at(y1, x0) * (1 - wx) + at(y1, x1) * wx) * wy


def _exact_flow(case, seed):
    h, w = case["h"], case["w"]
    window = _gaussian(5, 2.5)
    pyramids = []
    for rgb in _frames(case, seed, 2):
        c = rgb.to(torch.int64)
        f = ((77 * c[..., 0] + 150 * c[..., 1] + 29 * c[..., 2] + 128) >> 8).double() / 255.0
        levels = [f]
        for _ in range(case["levels"] - 1):
            levels.append(_filter(levels[-1], (1 / 16, 4 / 16, 6 / 16, 4 / 16, 1 / 16), 2)[::2, ::2].contiguous())
        pyramids.append([_expansion(v) for v in levels])
    d = None
    for e1, e2 in zip(reversed(pyramids[0]), reversed(pyramids[1])):
        lh, lw = e1.shape[1:]
        gy = torch.arange(lh, device=DEV, dtype=torch.float64)[:, None].expand(lh, lw)
        gx = torch.arange(lw, device=DEV, dtype=torch.float64)[None, :].expand(lh, lw)
        d = torch.zeros((2, lh, lw), dtype=torch.float64, device=DEV) if d is None else 2.0 * _bilinear(d, gy / 2, gx / 2)
        for _ in range(3):
            warped = _bilinear(e2, gy + d[1], gx + d[0])
            axx, axy, ayy = (0.5 * (e1[i] + warped[i]) for i in range(3))
            bx = -0.5 * (warped[3] - e1[3]) + axx * d[0] + axy * d[1]
            by = -0.5 * (warped[4] - e1[4]) + axy * d[0] + ayy * d[1]
            g11, g12, g22, h1, h2 = (_filter(t, window, 5) for t in (
                axx * axx + axy * axy, axy * (axx + ayy), axy * axy + ayy * ayy, axx * bx + axy * by, axy * bx + ayy * by))
            lam = 1e-4 + 1e-2 * 0.5 * (g11 + g22)
            m11, m22, r1, r2 = g11 + lam, g22 + lam, h1 + lam * d[0], h2 + lam * d[1]
            det = m11 * m22 - g12 * g12
            d = torch.stack([(m22 * r1 - g12 * r2) / det, (m11 * r2 - g12 * r1) / det])
    ys, xs = [i * h // 24 for i in range(25)], [i * w // 24 for i in range(25)]
    square = (d * d).sum(0)
    total = torch.zeros((h + 1, w + 1), dtype=torch.float64, device=DEV)
    total[1:, 1:] = square.cumsum(0).cumsum(1)
    corner = total[ys][:, xs]
    area = torch.tensor(np.diff(ys)[:, None] * np.diff(xs)[None, :], device=DEV, dtype=torch.float64)
    mean = (corner[1:, 1:] - corner[:-1, 1:] - corner[1:, :-1] + corner[:-1, :-1]) / area
    motion = mean.clamp(min=0).sqrt().reshape(-1)
    n_static = int((motion < 0.5).sum())
    redundant = int(np.float32(n_static) / np.float32(TOKENS) > np.float32(0.9))
    return {"uv": d, "motion": motion, "static_and_redundant": torch.tensor([n_static, redundant], dtype=torch.int32, device=DEV)}
