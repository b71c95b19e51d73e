"""The calls this library is used for, as timed cases.

A case is a dict of plain values: ``kind`` names the entry point --

* ``clip``   one ``Inpainter(frames, masks)`` call (FP32, BF16 or FP8; joint or decoupled
  attention; plain or overlapping embedding; masked or all queries),
* ``stream`` one ``stream_step``: the newest frame of each of several open streams whose
  memory of past frames is full,
* ``train``  one training step up to the gradients: ``load_params``, ``train_forward``,
  ``l1_loss``, ``train_backward`` (FP32 or bf16 products),
* ``camera`` ``prep_frame`` and ``post_frame`` around the network at camera resolution --

and the rest are the network's shape (``drsynth.NetCfg``) and the sizes.  Every input is made
from the seed on the GPU: frames of dark and bright textured surfaces that pan, private masks
of moving blobs covering a given share of each clip, weights N(0, 0.02^2).
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

import drsynth
from paper_2509_10466_amd import Inpainter
from paper_2509_10466_amd.api import flatten_params


def _net(name, **more):
    n = drsynth.NETS[name]
    return dict(dim=n.dim, heads=n.heads, blocks=n.blocks, mlp_ratio=n.mlp_ratio, win_h=n.win_h, win_w=n.win_w,
                win_t=n.win_t, attn="joint", overlap=False) | more


def _cfg(c):
    return drsynth.NetCfg(dim=c["dim"], heads=c["heads"], blocks=c["blocks"], mlp_ratio=c["mlp_ratio"], patch=4,
                          win_h=c["win_h"], win_w=c["win_w"], win_t=c["win_t"], attn=c["attn"], overlap=c["overlap"])


def _clip(net, B, H, W, precision="bf16", queries="masked", cover=0.26, **more):
    return _net(net, **more) | dict(kind="clip", B=B, H=H, W=W, precision=precision, queries=queries, cover=cover)


def _stream(net, n, H, W, slots=4, cover=0.26, **more):
    return _net(net, **more) | dict(kind="stream", n=n, H=H, W=W, slots=slots, cover=cover)


def _train(net, B, H, W, precision, cover=0.26, **more):
    return _net(net, **more) | dict(kind="train", B=B, H=H, W=W, precision=precision, cover=cover)


def _camera(H, W, instances, radius):
    return dict(kind="camera", H=H, W=W, instances=instances, radius=radius, cover=0.2)


def listed():
    return [
        # one small frame: the shortest call, set by launches and latency
        dict(name="tiny64_bf16", **_clip("tiny64", 1, 64, 64, cover=0.15)),
        # the headline clip, one call per clip
        dict(name="clip240_bf16", **_clip("clip240", 1, 240, 432)),
        # the same clip in plain FP32, the precision results are checked against
        dict(name="clip240_fp32", **_clip("clip240", 1, 240, 432, "fp32")),
        # the decoupled spatial/temporal network, two clips at a time
        dict(name="clip240_decoupled", **_clip("clip240", 2, 240, 432, attn="decoupled")),
        # every token a query (the whole frame regenerated) at the served resolution
        dict(name="clip480_all_queries", **_clip("clip240", 1, 480, 864, queries="all")),
        # 720p clips on the large network, BF16 and FP8
        dict(name="clip720_bf16", **_clip("clip720", 1, 720, 1280)),
        dict(name="clip720_fp8", **_clip("clip720", 1, 720, 1280, "fp8")),
        # one collaborator's frame: stream mode at its smallest
        dict(name="stream240_x1", **_stream("clip240", 1, 240, 432)),
        # a served batch of eight collaborators
        dict(name="stream480_x8", **_stream("clip240", 8, 480, 864)),
        # a training step in FP32 and with bf16 products
        dict(name="train240_fp32", **_train("clip240", 2, 240, 432, "fp32")),
        dict(name="train240_bf16", **_train("clip240", 4, 240, 432, "bf16")),
        # one camera frame's steps around the network
        dict(name="camera720", **_camera(720, 1280, 4, 5)),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more case: network width, depth, windows, resolution and batch drawn over the ranges
    of the listed ones (spread over the logarithm), none dearer than the dearest of them."""
    most = {"flops": {}, "bytes": 0.0}
    for c in listed():
        w = work(c)
        p = c.get("precision", "bf16")
        most["flops"][p] = max(most["flops"].get(p, 0.0), w["flops"])
        most["bytes"] = max(most["bytes"], w["bytes"])
    while True:
        kind = rng.choice(("clip",) * 5 + ("stream",) * 2 + ("train",) * 2 + ("camera",))
        if kind == "camera":
            return _camera(2 * _log_int(rng, 60, 360), 4 * _log_int(rng, 40, 320), rng.randint(0, 8), rng.randint(0, 12))
        dim = rng.choice((64, 128, 256, 256, 384))
        wh, ww, wt = rng.choice(((8, 8, 1), (5, 9, 5), (5, 9, 5), (6, 10, 5), (4, 7, 3)))  # the last in FP32 only
        net = dict(dim=dim, heads=dim // rng.choice((32, 64, 64)), blocks=rng.randint(1, 12), mlp_ratio=4, win_h=wh,
                   win_w=ww, win_t=wt, attn="joint", overlap=False)
        H, W = 4 * wh * _log_int(rng, 1, 30), 4 * ww * _log_int(rng, 1, 32)
        cover = round(rng.uniform(0.10, 0.40), 3)
        if kind == "clip":
            precision = rng.choice(("bf16", "bf16", "bf16", "fp32", "fp8"))
            if precision == "fp8" and dim % 128:
                precision = "bf16"
            if wt == 3:
                precision = "fp32"
            variant = rng.random()
            if precision != "fp32" and variant < 0.2 and wt > 1:
                net["attn"] = "decoupled"
            elif precision == "bf16" and variant > 0.8:
                net["overlap"] = True
            c = net | dict(kind=kind, B=rng.randint(1, 3), H=H, W=W, precision=precision,
                           queries="all" if rng.random() < 0.15 else "masked", cover=cover)
        elif kind == "stream":
            if wt != 5:
                continue
            c = net | dict(kind=kind, n=_log_int(rng, 1, 16), H=H, W=W, slots=rng.randint(0, wt - 1), cover=cover)
        else:
            c = net | dict(kind=kind, B=rng.randint(1, 4), H=H, W=W, precision=rng.choice(("fp32", "bf16")), cover=cover)
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"][c.get("precision", "bf16")]:
            return c


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------

def _noise(gen, T, H, W, cell, channels):
    """Smooth noise panning over T frames, [T, H, W, channels], about N(0, 1)."""
    gh, gw = -(-(H + 64) // cell) + 2, -(-(W + 64) // cell) + 2
    grid = torch.randn((1, channels, gh, gw), generator=gen, device="cuda")
    big = F.interpolate(grid, size=(gh * cell, gw * cell), mode="bicubic", align_corners=False)[0]
    vy, vx = (int(v) for v in torch.randint(1, 7, (2,), generator=gen, device="cuda").tolist())
    out = [big[:, t * vy % 64:t * vy % 64 + H, t * vx % 64:t * vx % 64 + W] for t in range(T)]
    return torch.stack(out).permute(0, 2, 3, 1)


def _video(gen, T, H, W, cover):
    """frames [T, H, W, 3] f32 in [0, 1] and masks [T, H, W] u8 covering ``cover`` of them."""
    tone = torch.where(_noise(gen, T, H, W, 48, 3) < 0, 0.2, 0.8)
    frames = (tone + 0.12 * torch.tanh(_noise(gen, T, H, W, 6, 3))).float().contiguous()
    blob = _noise(gen, T, H, W, max(8, min(48, H // 4)), 1)[..., 0].contiguous()
    k = max(1, int(round((1.0 - cover) * blob.numel())))
    level = blob.reshape(-1).sort().values[min(k, blob.numel() - 1)]
    return frames, (blob >= level).to(torch.uint8).contiguous()


def _inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    if c["kind"] == "camera":
        H, W = c["H"], c["W"]
        frames, mask = _video(gen, 1, H, W, c["cover"])
        rgb = (255.0 * frames[0]).to(torch.uint8)
        bgra = torch.cat([rgb[..., [2, 1, 0]], torch.full((H, W, 1), 255, dtype=torch.uint8, device="cuda")], -1).contiguous()
        K = c["instances"]
        band = torch.arange(W, device="cuda") * max(K, 1) // W
        inst = torch.stack([mask[0] * (band == k) for k in range(K)]).to(torch.uint8).contiguous() if K else None
        pred = torch.rand((H // 2, W // 2, 3), generator=gen, device="cuda")
        return bgra, inst, 0b10101, pred
    if c["kind"] == "stream":
        clips = [_video(gen, c["slots"] + 1, c["H"], c["W"], c["cover"]) for _ in range(c["n"])]
    else:
        clips = [_video(gen, c["win_t"], c["H"], c["W"], c["cover"]) for _ in range(c["B"])]
    return torch.stack([f for f, _ in clips]), torch.stack([m for _, m in clips])


def prepare(case, seed):
    c = case
    if c["kind"] == "camera":
        bgra, inst, select, pred = _inputs(c, seed)
        cfg = drsynth.NETS["tiny64"]
        return dict(case=c, eng=Inpainter(cfg, drsynth.make_weights(cfg, 0)), bgra=bgra, inst=inst, select=select, pred=pred)
    cfg = _cfg(c)
    weights = drsynth.make_weights(cfg, seed)
    eng = Inpainter(cfg, weights)
    frames, masks = _inputs(c, seed)
    s = dict(case=c, eng=eng, frames=frames, masks=masks)
    if c["kind"] == "clip":
        eng.reserve(c["B"], c["win_t"], c["H"], c["W"], c["precision"])
    elif c["kind"] == "stream":
        s["sids"] = [eng.stream_open(c["H"], c["W"], slots=c["slots"]) for _ in range(c["n"])]
        for t in range(c["slots"]):
            eng.stream_step(s["sids"], [f[t] for f in frames], [m[t] for m in masks])
        s["new"] = [f[-1].contiguous() for f in frames], [m[-1].contiguous() for m in masks]
    else:
        eng.train_precision(c["precision"])
        s["params"] = flatten_params(cfg, weights).cuda()
        s["cut"] = frames * (masks == 0)[..., None]
    return s


def run(state):
    c, eng = state["case"], state["eng"]
    if c["kind"] == "clip":
        return eng(state["frames"], state["masks"], c["precision"], c["queries"])
    if c["kind"] == "stream":
        return eng.stream_step(state["sids"], *state["new"])
    if c["kind"] == "train":
        eng.load_params(state["params"])
        pred, saved = eng.train_forward(state["cut"], state["masks"])
        loss, dpred = eng.l1_loss(pred, state["frames"], state["masks"])
        grads = eng.train_backward(saved, dpred)
        saved.close()
        return {"pred": pred, "loss": loss, "grads": grads}
    low, mask_low, mask_full = eng.prep_frame(state["bgra"], state["inst"], state["select"], c["radius"])
    return {"low": low, "mask_low": mask_low, "mask_full": mask_full,
            "out": eng.post_frame(state["bgra"], state["pred"], mask_full)}


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------

def work(case):
    """Bytes: every input and weight read once, every output written once.  Operations: with N
    tokens, the queries that the mask's share makes of them and the tokens of windows that
    have queries (about twice that share)."""
    c = case
    H, W = c["H"], c["W"]
    if c["kind"] == "camera":
        px = H * W
        return {"bytes": px * (4 + c["instances"] + 1 + 4) + px / 4 * (1 + 12 + 12) + px * 5, "flops": 0.0}
    C, R, L = c["dim"], c["mlp_ratio"] * c["dim"], c["blocks"]
    clips, T = (c["n"], 1) if c["kind"] == "stream" else (c["B"], c["win_t"])
    px = clips * T * H * W
    N = px / 16
    full = c.get("queries") == "all"
    nq = N if full else min(1.0, 1.12 * c["cover"]) * N
    na = N if full or c["kind"] == "stream" else min(1.0, 2 * c["cover"]) * N
    sf = c["win_h"] * c["win_w"]
    joint = sf * ((c["slots"] + 1) if c["kind"] == "stream" else c["win_t"])
    S = joint if c["attn"] == "joint" else 0.5 * (sf + joint / sf)
    k = 192 if c["overlap"] else 48
    weights = L * (4 * C * C + 2 * C * R) + 2 * C * k
    block = 2 * na * C * 2 * C + 4 * nq * C * C + 4 * nq * S * C + 4 * nq * C * R
    flops = L * block + 2 * N * k * C + 2 * (N if c["kind"] == "train" else nq) * k * C
    size = {"fp32": 4, "bf16": 2, "fp8": 1}[c.get("precision", "bf16")]
    if c["kind"] == "train":
        return {"bytes": px * (12 + 1) * 2 + px * 12 + weights * 4 * 3, "flops": 3 * flops}
    moved = px * (12 + 1 + 12) + weights * size
    if c["kind"] == "stream":  # the remembered keys and values read, the new frame's written
        moved += L * N * 2 * C * 2 * (c["slots"] + 1)
    return {"bytes": moved, "flops": flops}


# ------------------------------------------------------------------------------------------
# the same results in 64 bits, from torch's own operations
# ------------------------------------------------------------------------------------------

def _split(x, c, kind):
    """[B, T, h, w, C] -> [groups, tokens of a group, C] of one attention kind."""
    B, T, h, w, C = x.shape
    wt, wh, ww = c["win_t"] if kind != "spatial" else 1, c["win_h"], c["win_w"]
    if kind == "temporal":
        wh = ww = 1
    x = x.reshape(B, T // wt, wt, h // wh, wh, w // ww, ww, C).permute(0, 1, 3, 5, 2, 4, 6, 7)
    return x.reshape(-1, wt * wh * ww, C)


def _join(x, c, kind, shape):
    B, T, h, w, C = shape
    wt, wh, ww = c["win_t"] if kind != "spatial" else 1, c["win_h"], c["win_w"]
    if kind == "temporal":
        wh = ww = 1
    x = x.reshape(B, T // wt, h // wh, w // ww, wt, wh, ww, C).permute(0, 1, 4, 2, 5, 3, 6, 7)
    return x.reshape(shape)


def _attend(q, k, v, heads, chunk):
    """softmax(q k^T / sqrt(dh)) v per head over [groups, tokens, C], ``chunk`` groups at a time."""
    dh = q.shape[-1] // heads
    out = []
    for i in range(0, q.shape[0], chunk):
        a, b, d = (t[i:i + chunk].reshape(-1, t.shape[1], heads, dh).transpose(1, 2).contiguous() for t in (q, k, v))
        p = torch.softmax(a @ b.transpose(2, 3).contiguous() / math.sqrt(dh), -1)
        out.append((p @ d).transpose(1, 2).reshape(-1, q.shape[1], heads * dh))
    return torch.cat(out)


def _flags(masks, c):
    B, T, H, W = masks.shape
    m = (masks != 0).double().reshape(B * T, 1, H, W)
    f = F.max_pool2d(m, 8, 4, 2) if c["overlap"] else F.max_pool2d(m, 4)
    return f.reshape(B, T, H // 4, W // 4) > 0


def _embed(frames, masks, P, c):
    B, T, H, W, _ = frames.shape
    img = (frames * (masks == 0)[..., None]).reshape(B * T, H, W, 3).permute(0, 3, 1, 2)
    k, pad = (8, 2) if c["overlap"] else (4, 0)
    cols = F.unfold(img, k, padding=pad, stride=4).transpose(1, 2)
    return (cols @ P["embed.w"].reshape(c["dim"], -1).T + P["embed.b"]).reshape(B, T, H // 4, W // 4, c["dim"])


def _decode(x, P, c):
    B, T, h, w, C = x.shape
    z = F.layer_norm(x, (C,), P["lnf.g"], P["lnf.b"], 1e-5).reshape(B * T, h * w, C)
    k, pad = (8, 2) if c["overlap"] else (4, 0)
    y = F.fold((z @ P["dec.w"].reshape(C, -1)).transpose(1, 2), (4 * h, 4 * w), k, padding=pad, stride=4)
    y = y + P["dec.b"][:, None, None]
    return torch.sigmoid(y).permute(0, 2, 3, 1).reshape(B, T, 4 * h, 4 * w, 3)


def _mlp(x, o, P, l, C):
    x = x + o @ P[f"blk{l}.wo"].T + P[f"blk{l}.bo"]
    u = F.layer_norm(x, (C,), P[f"blk{l}.ln2.g"], P[f"blk{l}.ln2.b"], 1e-5)
    return x + F.gelu(u @ P[f"blk{l}.w1"].T + P[f"blk{l}.b1"]) @ P[f"blk{l}.w2"].T + P[f"blk{l}.b2"]


def _qkv(x, P, l, C):
    u = F.layer_norm(x, (C,), P[f"blk{l}.ln1.g"], P[f"blk{l}.ln1.b"], 1e-5)
    return [u @ P[f"blk{l}.w{n}"].T + P[f"blk{l}.b{n}"] for n in "qkv"]


def _kind(c, l):
    return "joint" if c["attn"] == "joint" else ("spatial" if l % 2 == 0 else "temporal")


def _predict(frames, masks, P, c, chunk=256):
    """The decoder's output at every pixel of the clips."""
    C = c["dim"]
    x = _embed(frames, masks, P, c)
    update = torch.ones_like(_flags(masks, c)) if c.get("queries") == "all" else _flags(masks, c)
    for l in range(c["blocks"]):
        kind = _kind(c, l)
        many = chunk if kind != "temporal" else 1 << 16
        q, k, v = (_split(t, c, kind) for t in _qkv(x, P, l, C))
        o = _join(_attend(q, k, v, c["heads"], many), c, kind, x.shape)
        x = torch.where(update[..., None], _mlp(x, o, P, l, C), x)
    return _decode(x, P, c)


def _stream_frames(frames, masks, P, c):
    """The newest frame's prediction of streams that saw all of ``frames`` [n, slots + 1, ...]."""
    C = c["dim"]
    one = c | dict(win_t=1)
    past = [[] for _ in range(c["blocks"])]
    for t in range(frames.shape[1]):
        f, m = frames[:, t:t + 1], masks[:, t:t + 1]
        x = _embed(f, m, P, c)
        update = _flags(m, c)
        for l in range(c["blocks"]):
            kind = _kind(c, l)
            split = "temporal" if kind == "temporal" else "joint"
            q, k, v = (_split(a, one, split) for a in _qkv(x, P, l, C))
            seen = [] if kind == "spatial" else past[l]
            keys, vals = torch.cat([a for a, _ in seen] + [k], 1), torch.cat([b for _, b in seen] + [v], 1)
            o = _join(_attend(q, keys, vals, c["heads"], 512 if split == "joint" else 1 << 16), one, split, x.shape)
            x = torch.where(update[..., None], _mlp(x, o, P, l, C), x)
            past[l].append((k, v))
    return _decode(x, P, c)


def exact(case, seed):
    c = case
    if c["kind"] == "camera":
        bgra, inst, select, pred = _inputs(c, seed)
        H, W, r = c["H"], c["W"], c["radius"]
        union = torch.zeros((H, W), dtype=torch.float64, device="cuda")
        for k in range(c["instances"]):
            if select >> k & 1:
                union = torch.maximum(union, (inst[k] != 0).double())
        full = F.max_pool2d(union[None], 2 * r + 1, 1, r)[0]
        low = (bgra[..., [2, 1, 0]].double() / 255.0).reshape(H // 2, 2, W // 2, 2, 3).mean((1, 3))
        byte = torch.clamp(torch.round(255.0 * pred), 0, 255).repeat_interleave(2, 0).repeat_interleave(2, 1)
        out = torch.where(full[..., None] > 0, torch.cat([byte[..., [2, 1, 0]], bgra[..., 3:].float()], -1), bgra.float())
        return {"low": low, "mask_low": F.max_pool2d(full[None], 2)[0].to(torch.uint8), "mask_full": full.to(torch.uint8),
                "out": out.to(torch.uint8)}
    cfg = _cfg(c)
    P = {n: torch.from_numpy(np.asarray(a)).cuda().double() for n, a in drsynth.make_weights(cfg, seed).items()}
    frames, masks = _inputs(c, seed)
    x = frames.double()
    if c["kind"] == "clip":
        return torch.where((masks != 0)[..., None], _predict(x, masks, P, c), x)
    if c["kind"] == "stream":
        out = torch.where((masks[:, -1] != 0)[..., None], _stream_frames(x, masks, P, c)[:, 0], x[:, -1])
        return [o for o in out]
    P = {n: a.requires_grad_(True) for n, a in P.items()}
    pred = _predict(x, masks, P, c)
    inside = (masks != 0)[..., None].expand_as(x)
    off = (pred - x).abs()
    loss = sum(w * off[m].mean() for w, m in ((1.0, inside), (0.1, ~inside)) if bool(m.any()))
    names = [n for n, _ in drsynth.weight_order(cfg)]
    grads = torch.autograd.grad(loss, [P[n] for n in names])
    return {"pred": pred.detach(), "loss": loss.detach().reshape(1), "grads": torch.cat([g.reshape(-1) for g in grads])}
