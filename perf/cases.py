"""The work that a user of the package has it do, as cases that can be timed and compared.

Every case goes through the package's public entry points on inputs made on the GPU from a seed. The
scenes stand in for a walk around a loop: a camera at 1.5 m height between walls, revisits within about
2 m and 45 degrees, three latent frames per chunk. q, k and v are N(0, 1), as normalised attention
inputs are. A case is a dict of plain values whose "kind" says which entry point it calls.
"""

import math

import numpy as np
import torch

import paper_2607_21848_amd as rv

DEV = "cuda:0"
F = 3  # latent frames per chunk
SIGMA, LAM, EPS, DELTA = 2.0, 1.0, 0.05, 3
TAU_V, W_V = math.radians(45.0), 0.5
ROPE_PAIRS, THETA = 22, 10000.0
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}


def listed():
    return [
        # the tiny fp32 problem a program checks itself with: launch and latency only
        {"name": "attn_f32_tiny", "kind": "attn", "dtype": "f32", "h": 8, "w": 8, "frames": 1, "kv": 4, "ret": 2,
         "H": 1, "D": 64},
        # one layer of the Wan-1.3B loop closure (two retrieved chunks) in fp32, as a reference run takes it
        {"name": "attn_f32_wan13b", "kind": "attn", "dtype": "f32", "h": 30, "w": 52, "frames": 3, "kv": 18, "ret": 6,
         "H": 12, "D": 128},
        # one layer of a half-resolution preview (416 x 240): few queries, the chip is not filled by them alone
        {"name": "attn_bf16_preview", "kind": "attn", "dtype": "bf16", "h": 15, "w": 26, "frames": 3, "kv": 18,
         "ret": 6, "H": 12, "D": 128},
        # the Wan-1.3B loop closure with fp8 logits
        {"name": "attn_fp8_wan13b", "kind": "attn", "dtype": "fp8", "h": 30, "w": 52, "frames": 3, "kv": 18, "ret": 6,
         "H": 12, "D": 128},
        # one layer at 720p with the 14B model's 40 heads, the largest attention of the configurations
        {"name": "attn_bf16_wan14b", "kind": "attn", "dtype": "bf16", "h": 45, "w": 80, "frames": 3, "kv": 18,
         "ret": 6, "H": 40, "D": 128},
        # a whole chunk step over a history bank: top-4 retrieval, correspondence into 12 frames, attention
        {"name": "chunk_wan13b", "kind": "chunk", "dtype": "bf16", "h": 30, "w": 52, "p": 2, "bank": 200, "k": 4,
         "H": 12, "D": 128},
        # retrieval over an hour-long session's bank, and over a large archive for several queries
        {"name": "retrieve_session", "kind": "retrieve", "bank": 3000, "queries": 1, "k": 4},
        {"name": "retrieve_archive", "kind": "retrieve", "bank": 1000003, "queries": 4, "k": 8},
        # correspondence of many chunks at once (offline), with depth and between cameras sharing a centre
        {"name": "reproject_batch", "kind": "reproject", "B": 1024, "S": 6, "h": 30, "w": 52, "p": 2},
        {"name": "rotation_batch", "kind": "rotation", "B": 1024, "S": 6, "h": 30, "w": 52, "p": 2},
        # four retrieved chunks of eight layers reinstated in the cache
        {"name": "pack_wan13b", "kind": "pack", "dtype": "bf16", "layers": 8, "store": 12, "slots": 4, "h": 30,
         "w": 52, "H": 12, "D": 128},
        # one chunk of a running stream: ring, retrieval, correspondence, packing, every layer's attention
        {"name": "stream_wan13b", "kind": "stream", "dtype": "bf16", "layers": 8, "h": 30, "w": 52, "p": 2, "H": 12,
         "D": 128, "capacity": 8},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "chunk", "retrieve", "reproject", "rotation", "pack", "stream"])
    if kind == "attn":
        dtype = rng.choice(["f32", "bf16", "bf16", "fp8"])
        most = 4e11 if dtype == "f32" else 1.2e13
        while True:
            c = {"kind": kind, "dtype": dtype, "h": _log(rng, 5, 45), "w": _log(rng, 7, 80), "frames": F,
                 "kv": F * rng.randint(1, 10), "ret": 0, "H": _log(rng, 1, 40),
                 "D": rng.choice([64, 128]) if dtype == "f32" else 128}
            c["ret"] = F * rng.randint(0, min(4, c["kv"] // F - 1)) if c["kv"] > F else 0
            if _attn_flops(c) <= most:
                return c
    if kind == "chunk":
        return {"kind": kind, "dtype": rng.choice(["bf16", "fp8"]), "h": _log(rng, 8, 45), "w": _log(rng, 12, 80),
                "p": rng.choice([1, 2]), "bank": _log(rng, 50, 400), "k": rng.randint(1, 4), "H": _log(rng, 1, 16),
                "D": 128}
    if kind == "retrieve":
        bank = _log(rng, 30, 2000000)
        return {"kind": kind, "bank": bank, "queries": _log(rng, 1, 16), "k": _log(rng, 1, 32)}
    if kind in ("reproject", "rotation"):
        return {"kind": kind, "B": _log(rng, 1, 512), "S": F * rng.randint(1, 4), "h": _log(rng, 8, 45),
                "w": _log(rng, 12, 80), "p": rng.choice([1, 2])}
    h, w = _log(rng, 6, 30), _log(rng, 8, 52)
    if kind == "pack":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "layers": _log(rng, 1, 12),
                "store": rng.randint(4, 12), "slots": rng.randint(1, 4), "h": h, "w": w, "H": _log(rng, 1, 12),
                "D": 128}
    return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "layers": _log(rng, 1, 8),
            "h": h, "w": w, "p": rng.choice([1, 2]), "H": _log(rng, 1, 12), "D": 128, "capacity": rng.randint(6, 10)}


# ---- inputs ---------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _normal(g, dtype, *shape):
    if dtype == "fp8":
        return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32).to(torch.float8_e4m3fn)
    return torch.randn(*shape, generator=g, device=DEV, dtype=DTYPES[dtype])


def _pose(c, yaw, pitch):
    """Camera-to-world matrices [..., 4, 4] of cameras at c looking along yaw, pitched down by pitch."""
    cy, sy, cp, sp = yaw.cos(), yaw.sin(), pitch.cos(), pitch.sin()
    z = torch.zeros_like(yaw)
    fwd = torch.stack([cy * cp, sy * cp, -sp], -1)
    right = torch.stack([sy, -cy, z], -1)
    down = torch.linalg.cross(fwd, right)
    m = torch.zeros(*yaw.shape, 4, 4, device=DEV, dtype=torch.float64)
    m[..., :3, 0], m[..., :3, 1], m[..., :3, 2], m[..., :3, 3] = right, down, fwd, c
    m[..., 3, 3] = 1.0
    return m


def _loop(g, at, per_lap, radius):
    """Poses at the loop positions `at` (in chunks): heading along the tangent, 10 degrees of jitter."""
    th = 2.0 * math.pi * at / per_lap
    c = torch.stack([radius * th.cos(), radius * th.sin(), torch.full_like(th, 1.5)], -1)
    return _pose(c, th + math.pi / 2 + _uniform(g, -math.radians(10), math.radians(10), *at.shape),
                 torch.full_like(th, 0.08))


def _walls(g, n, radius):
    th = _uniform(g, 0.0, 2 * math.pi, n)
    normals = torch.stack([th.cos(), th.sin(), torch.zeros_like(th)], -1)
    ground = torch.tensor([[0.0, 0.0, 1.0]], device=DEV, dtype=torch.float64)
    return torch.cat([ground, normals]), torch.cat([torch.zeros(1, device=DEV, dtype=torch.float64),
                                                    radius + _uniform(g, 5.0, 25.0, n)])


def _intrinsics(h, w, p, *shape):
    """(fx, fy, cx, cy) of a 90 degree field of view, in depth pixels."""
    k = torch.tensor([w * p / 2.0, w * p / 2.0, w * p / 2.0, h * p / 2.0], device=DEV, dtype=torch.float32)
    return k.expand(*shape, 4).contiguous()


def _depth(g, c2w, h, w, p, walls):
    """Planar depth [..., h p, w p] of the walls seen from c2w, with 1% noise and a few empty pixels."""
    H, W = h * p, w * p
    K = _intrinsics(h, w, p).double()
    y, x = torch.meshgrid(torch.arange(H, device=DEV) + 0.5, torch.arange(W, device=DEV) + 0.5, indexing="ij")
    ray = torch.stack([(x - K[2]) / K[0], (y - K[3]) / K[1], torch.ones_like(x)], -1).float().reshape(-1, 3)
    flat = c2w.reshape(-1, 4, 4).float()
    out = torch.full((flat.shape[0], H * W), 50.0, device=DEV)
    for n, d in zip(*(v.float() for v in walls)):
        t = (d - flat[:, :3, 3] @ n)[:, None] / ((flat[:, :3, :3].transpose(1, 2) @ n) @ ray.T)
        out = torch.minimum(out, torch.where(t > 0, t, 50.0))
    out = out.clamp(0.5, 50.0) * (1.0 + 0.01 * torch.randn(out.shape, generator=g, device=DEV))
    out[torch.rand(out.shape, generator=g, device=DEV) < 0.005] = 0.0
    return out.reshape(*c2w.shape[:-2], H, W)


def _corr(g, S, frames, h, w):
    """A correspondence map into S frames: every token moved by its frame's shift, 10% of them occluded."""
    y, x = torch.meshgrid(torch.arange(h, device=DEV) + 0.5, torch.arange(w, device=DEV) + 0.5, indexing="ij")
    tok = torch.stack([x, y], -1).reshape(1, 1, h * w, 2)
    span = torch.tensor([w, h], device=DEV, dtype=torch.float32)
    shift = (torch.rand(S, frames, 1, 2, generator=g, device=DEV) - 0.5) * 0.4 * span
    uv = (tok + shift + 0.3 * torch.randn(S, frames, h * w, 2, generator=g, device=DEV)).reshape(S, -1, 2).contiguous()
    on = (uv >= 0).all(-1) & (uv < span).all(-1)
    idx = uv[..., 1].floor().int() * w + uv[..., 0].floor().int()
    idx = torch.where(on, idx, torch.full_like(idx, -3))
    hidden = (torch.rand(idx.shape, generator=g, device=DEV) < 0.1) & on
    return uv, torch.where(hidden, torch.full_like(idx, -4), idx).contiguous()


def _slots(kv, ret):
    """Retrieved frames sit behind the anchor chunk; every other frame is unbiased."""
    slot = torch.full((kv,), -1, dtype=torch.int32)
    at = min(F, kv - ret)
    slot[at:at + ret] = torch.arange(ret, dtype=torch.int32)
    return slot.to(DEV)


def _bank(g, bank, queries):
    """A bank on a loop 0.63 m per chunk, up to sixteen laps when long, and queries on the next lap."""
    lap = min(bank, max(200, bank // 16))
    radius = 0.1 * lap
    at = torch.arange(bank, device=DEV, dtype=torch.float64)
    chunk = bank + 25 * torch.arange(queries, device=DEV)
    return {"bank": _loop(g, at % lap, lap, radius).float(), "query": _loop(g, chunk.double() % lap, lap, radius).float(),
            "chunk": chunk.int(), "lap": lap, "radius": radius, "E": 2.0 * radius, "tau_c": 2.0 / (2.0 * radius)}


def _attn_inputs(g, c, frames, kv, S):
    hw = c["h"] * c["w"]
    vdt = "bf16" if c["dtype"] == "fp8" else c["dtype"]
    return {"q": _normal(g, c["dtype"], frames * hw, c["H"], c["D"]), "k": _normal(g, c["dtype"], kv * hw, c["H"], c["D"]),
            "v": _normal(g, vdt, kv * hw, c["H"], c["D"]), "slot": _slots(kv, S)}


def prepare(case, seed):
    g, c = _gen(seed), case
    s = {"case": c}
    if c["kind"] == "attn":
        s.update(_attn_inputs(g, c, c["frames"], c["kv"], c["ret"]))
        s["uv"], s["idx"] = _corr(g, c["ret"], c["frames"], c["h"], c["w"]) if c["ret"] else (None, None)
    elif c["kind"] == "retrieve":
        s.update(_bank(g, c["bank"], c["queries"]))
    elif c["kind"] == "chunk":
        s.update(_bank(g, c["bank"], 1))
        h, w, p, n = c["h"], c["w"], c["p"], c["bank"]
        walls = _walls(g, 16, s["radius"])
        frames = _loop(g, torch.arange(n * F, device=DEV, dtype=torch.float64) / F, s["lap"], s["radius"])
        target = _loop(g, (n * F + torch.arange(F, device=DEV, dtype=torch.float64)) / F % s["lap"], s["lap"], s["radius"])
        s["bank"], s["query"] = frames[F // 2::F].float().contiguous(), target[F // 2][None].float().contiguous()
        s["src"] = (_depth(g, frames, h, w, p, walls), frames.float(), _intrinsics(h, w, p, n * F))
        s["tgt"] = (_depth(g, target[None], h, w, p, walls), target[None].float(), _intrinsics(h, w, p, 1, F))
        S = c["k"] * F
        s.update(_attn_inputs(g, c, F, S + 4 * F, S))
        # a serving loop keeps its outputs and its workspace
        Lq, vdt = F * h * w, s["v"].dtype
        s["out_r"] = (torch.empty(1, c["k"], dtype=torch.int32, device=DEV), torch.empty(1, c["k"], device=DEV),
                      torch.empty(1, dtype=torch.int32, device=DEV), torch.empty(1, S, dtype=torch.int32, device=DEV))
        s["out_c"] = (torch.empty(1, S, Lq, 2, device=DEV), torch.empty(1, S, Lq, dtype=torch.int32, device=DEV))
        s["out_a"] = (torch.empty(Lq, c["H"], c["D"], dtype=vdt, device=DEV), torch.empty(c["H"], Lq, device=DEV))
        ws = rv.attention_workspace_size(s["q"].dtype, Lq, s["k"].shape[0], c["H"], c["D"])
        s["ws"] = torch.empty(max(ws, 16), dtype=torch.uint8, device=DEV)
    elif c["kind"] == "reproject":
        B, S, h, w, p = (c[n] for n in ("B", "S", "h", "w", "p"))
        walls = _walls(g, 16, 20.0)
        th = _uniform(g, 0.0, 2 * math.pi, B, 1)
        at = th + 0.5 / 20.0 * torch.arange(S, device=DEV)  # the stored frames, 0.5 m apart
        ring = lambda a: torch.stack([20 * a.cos(), 20 * a.sin(), torch.full_like(a, 1.5)], -1)  # noqa: E731
        src = _pose(ring(at), at + math.pi / 2, torch.full_like(at, 0.05))
        tgt = _pose(ring(at[:, :F]) + _uniform(g, -0.17, 0.17, B, F, 3),
                    at[:, :F] + math.pi / 2 + _uniform(g, -math.radians(5), math.radians(5), B, F),
                    0.05 + _uniform(g, -math.radians(2), math.radians(2), B, F))
        s["tgt"] = (_depth(g, tgt, h, w, p, walls), tgt.float(), _intrinsics(h, w, p, B, F))
        s["src"] = (_depth(g, src, h, w, p, walls), src.float(), _intrinsics(h, w, p, B, S))
    elif c["kind"] == "rotation":
        # turning in place by 90 to 180 degrees (even problems), or zooming from 90 to 35 degrees (odd ones), and back
        B, S, h, w, p = (c[n] for n in ("B", "S", "h", "w", "p"))
        centre = _uniform(g, -20.0, 20.0, B, 1, 3).float().double()
        even = (torch.arange(B, device=DEV) % 2 == 0)[:, None]
        leg = torch.arange(S, device=DEV, dtype=torch.float64) / max(S - 1, 1)
        yaw = _uniform(g, 0.0, 2 * math.pi, B, 1) + torch.where(even, _uniform(g, math.pi / 2, math.pi, B, 1), 0.0) * leg
        fov = torch.where(even, 90.0, 90.0 - 55.0 * leg)
        pick = torch.randint(0, S, (B, F), generator=g, device=DEV)
        K = _intrinsics(h, w, p, B, S).clone()
        K[..., :2] *= (1.0 / torch.tan(torch.deg2rad(fov) / 2))[..., None].float()
        s["src"] = (_pose(centre, yaw, torch.full_like(yaw, 0.05)).float(), K)
        s["tgt"] = (_pose(centre, yaw.gather(1, pick) + _uniform(g, -0.17, 0.17, B, F),
                          0.05 + _uniform(g, -0.05, 0.05, B, F)).float(),
                    K.gather(1, pick[..., None].expand(B, F, 4)).contiguous())
    elif c["kind"] == "pack":
        T, row = F * c["h"] * c["w"], (c["H"], c["D"])
        s["store"] = [_normal(g, c["dtype"], c["layers"], c["store"], T, *row) for _ in range(2)]
        s["cache"] = [torch.zeros(c["layers"], (c["slots"] + 4) * T, *row, dtype=DTYPES[c["dtype"]], device=DEV) for _ in range(2)]
        s["sel"] = torch.randperm(c["store"], generator=g, device=DEV)[:c["slots"]].int()
    else:
        # a stream that has left its anchor and stands where it stood a ring ago: every later step has the same result
        h, w, p, n = c["h"], c["w"], c["p"], c["layers"]
        walls = _walls(g, 12, 4.0)
        poses = _loop(g, torch.arange(2 * F, device=DEV, dtype=torch.float64).reshape(2, F) / F, 8.0, 4.0)
        K = _intrinsics(h, w, p, F)
        shape = (n, F * h * w, c["H"], c["D"])
        s["chunks"] = [(_depth(g, m, h, w, p, walls), m.float().contiguous(), K, *[_normal(g, c["dtype"], *shape) for _ in range(3)])
                       for m in poses]
        s["driver"] = rv.StreamDriver(F=F, h=h, w=w, p=p, H=c["H"], D=c["D"], layers=n, dtype=DTYPES[c["dtype"]],
                                      capacity=c["capacity"], max_chunks=1 << 16, E=8.0, w_v=W_V, tau_c=0.25, tau_v=TAU_V,
                                      delta=DELTA, eps=EPS, lam=LAM, sigma=SIGMA, softmax_scale=c["D"] ** -0.5,
                                      rope_t_pairs=ROPE_PAIRS, rope_theta=THETA)
        for i in range(c["capacity"] + 4):
            s["driver"].step(*s["chunks"][min(i, 1)])
    return s


# ---- one pass -------------------------------------------------------------


def _retrieve(s, k, frames=None, out=None):
    return rv.retrieve_chunks(s["bank"], s["query"], s["chunk"], E=s["E"], w_v=W_V, tau_c=s["tau_c"], tau_v=TAU_V,
                              delta=DELTA, first_candidate=1, k=k, frames_per_chunk=frames, out=out)


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "attn":
        return rv.biased_chunk_attention(s["q"], s["k"], s["v"], s["slot"], s["uv"], s["idx"], h=c["h"], w=c["w"],
                                         softmax_scale=c["D"] ** -0.5, lam=LAM, sigma=SIGMA)
    if c["kind"] == "retrieve":
        return _retrieve(s, c["k"], F)
    if c["kind"] == "chunk":
        idx, score, count, sel = _retrieve(s, c["k"], F, s["out_r"])
        uv, code = rv.reproject_correspondence(*s["tgt"], *s["src"], p=c["p"], eps=EPS, src_sel=sel, out=s["out_c"])
        o, lse = rv.biased_chunk_attention(s["q"], s["k"], s["v"], s["slot"], uv[0], code[0], h=c["h"], w=c["w"],
                                           softmax_scale=c["D"] ** -0.5, lam=LAM, sigma=SIGMA, out=s["out_a"],
                                           workspace=s["ws"])
        return idx, score, count, uv, code, o, lse
    if c["kind"] == "reproject":
        return rv.reproject_correspondence(*s["tgt"], *s["src"], p=c["p"], eps=EPS)
    if c["kind"] == "rotation":
        return rv.reproject_rotation(*s["tgt"], *s["src"], h=c["h"], w=c["w"], p=c["p"])
    if c["kind"] == "pack":
        T = F * c["h"] * c["w"]
        rv.pack_retrieved_kv(*s["store"], s["sel"], *s["cache"], F=F, h=c["h"], w=c["w"], dst_pos=F, dst_row0=T,
                             rope_t_pairs=ROPE_PAIRS, rope_theta=THETA)
        return tuple(s["cache"])
    return s["driver"].step(*s["chunks"][1])


# ---- what a pass cannot do without ----------------------------------------

SIZE = {"f32": 4, "bf16": 2, "fp8": 1}


def _attn_flops(c):
    hw = c["h"] * c["w"]
    return 4.0 * c["frames"] * c["kv"] * hw * hw * c["H"] * c["D"]


def _attn_work(c, frames, kv, S):
    hw, e = c["h"] * c["w"], SIZE[c["dtype"]]
    ve = 2 if c["dtype"] == "fp8" else e
    row = c["H"] * c["D"]
    return {"bytes": hw * row * (frames * (e + ve) + kv * (e + ve)) + 4 * c["H"] * frames * hw + 12 * S * frames * hw,
            "flops": _attn_flops(dict(c, frames=frames, kv=kv))}


def _reproject_work(c, B, S):
    """Both depth maps read, a position and a code written per pair; about 40 operations per pair."""
    hw = c["h"] * c["w"]
    return {"bytes": B * hw * (4 * (F + S) * c["p"] ** 2 + 12 * F * S), "flops": 40.0 * B * F * S * hw}


def work(case):
    c = case
    if c["kind"] == "attn":
        return _attn_work(c, c["frames"], c["kv"], c["ret"])
    if c["kind"] == "retrieve":
        return {"bytes": 64 * (c["bank"] + c["queries"]) + c["queries"] * c["k"] * (8 + 4 * F),
                "flops": 20.0 * c["bank"] * c["queries"]}
    if c["kind"] == "chunk":
        S = c["k"] * F
        a, b = _attn_work(c, F, S + 4 * F, S), _reproject_work(c, 1, S)
        return {"bytes": a["bytes"] + b["bytes"] + 64 * c["bank"], "flops": a["flops"] + b["flops"]}
    if c["kind"] == "reproject":
        return _reproject_work(c, c["B"], c["S"])
    if c["kind"] == "rotation":
        n = c["B"] * F * c["S"] * c["h"] * c["w"]
        return {"bytes": 12 * n, "flops": 20.0 * n}
    image = F * c["h"] * c["w"] * c["H"] * c["D"] * SIZE[c["dtype"]]  # one layer's keys (or values) of a chunk
    if c["kind"] == "pack":
        return {"bytes": 4 * c["layers"] * c["slots"] * image, "flops": 0}
    # the chunk's q, k and v read, o written, k and v kept, four earlier parts' keys and values read
    a = _attn_work(c, F, 5 * F, F)
    return {"bytes": c["layers"] * (6 * image + 2 * 4 * image), "flops": c["layers"] * a["flops"]}


def tolerance(case):
    """Choices, codes, positions and copied or once-rounded bytes are the same bit for bit; attention rounds."""
    if case["kind"] in ("retrieve", "reproject", "rotation", "pack"):
        return "exact"
    # fp32 sums in another order: 2.7e-6 against 64 bits over 28080 keys; bf16: the probabilities and the result are
    # rounded to bf16 once each (2.4e-3 against 64 bits)
    return {"rel": 1e-5, "max": 1e-3} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.2}


# ---- the same in 64 bits --------------------------------------------------


def _exact_attention(q, k, v, slot, uv, idx, h, w, scale):
    """o [Lq, H, D] and lse [H, Lq] in double, one head and a block of queries at a time."""
    Lq, H, D = q.shape
    hw, S = h * w, 0 if uv is None else uv.shape[0]
    wide = lambda x: (x.float() if x.dtype == torch.float8_e4m3fn else x).double()  # noqa: E731
    key = torch.arange(hw, device=DEV)
    at = torch.stack([key % w + 0.5, key // w + 0.5], -1).double()
    o, lse = torch.empty(Lq, H, D, device=DEV, dtype=torch.float64), torch.empty(H, Lq, device=DEV, dtype=torch.float64)
    step = max(1, (1 << 27) // k.shape[0])
    frame_of = slot.tolist()
    for hd in range(H):
        kh, vh = wide(k[:, hd]).t().contiguous(), wide(v[:, hd]).contiguous()
        for r in range(0, Lq, step):
            a = (wide(q[r:r + step, hd]) @ kh).mul_(scale)
            for f, sl in enumerate(frame_of):
                if 0 <= sl < S:
                    u = uv[sl, r:r + step].double()
                    d = -((at[None, :, 0] - u[:, None, 0]) ** 2 + (at[None, :, 1] - u[:, None, 1]) ** 2) / (2 * SIGMA ** 2)
                    a[:, f * hw:(f + 1) * hw] += torch.where((idx[sl, r:r + step] >= 0)[:, None], LAM * d, 0.0)
            m = a.amax(1, keepdim=True)
            a = a.sub_(m).exp_()
            l = a.sum(1, keepdim=True)
            o[r:r + step, hd] = (a @ vh) / l
            lse[hd, r:r + step] = (m + l.log())[:, 0]
    return o, lse


def _exact_retrieve(s, k):
    b, q = s["bank"].double(), s["query"].double()
    N, Q = b.shape[0], q.shape[0]
    idx = torch.full((Q, k), -1, device=DEV, dtype=torch.int32)
    score = torch.full((Q, k), math.inf, device=DEV, dtype=torch.float64)
    count = torch.zeros(Q, device=DEV, dtype=torch.int32)
    j = torch.arange(N, device=DEV)
    E, tau = (float(np.float32(s[n])) for n in ("E", "tau_c"))
    cos_v = math.cos(float(np.float32(TAU_V)))
    for i in range(Q):
        x = b[:, :3, 3] - q[i, :3, 3]
        d = torch.sqrt(x[:, 0] * x[:, 0] + x[:, 1] * x[:, 1] + x[:, 2] * x[:, 2]) / E
        v, u = b[:, :3, 2], q[i, :3, 2]
        al = v[:, 0] * u[0] + v[:, 1] * u[1] + v[:, 2] * u[2]
        ok = (j >= 1) & (int(s["chunk"][i]) - j >= DELTA) & (d <= tau) & (al >= cos_v)
        sc, order = torch.sort(torch.where(ok, d + W_V * (1.0 - al), math.inf), stable=True)
        n = min(k, int(ok.sum()))
        idx[i, :n], score[i, :n], count[i] = order[:n].int(), sc[:n], n
    sel = (idx.repeat_interleave(F, 1) * F + torch.arange(F, device=DEV).repeat(k)).int()
    return idx, score, count, torch.where(idx.repeat_interleave(F, 1) >= 0, sel, torch.full_like(sel, -1))


def _exact_reproject(tgt, src, h, w, p, sel=None):
    """uv [B, S, Tq h w, 2] in double and codes [B, S, Tq h w], one problem at a time."""
    pool = lambda d: d.double().reshape(*d.shape[:-2], h, p, w, p).mean((-1, -3)).reshape(*d.shape[:-2], h * w)  # noqa: E731
    (td, tm, tk), (sd, sm, sk) = tgt, src
    B, Tq = td.shape[:2]
    S = sd.shape[1] if sel is None else sel.shape[1]
    t = torch.arange(h * w, device=DEV)
    ux, uy = (t % w).double() + 0.5, (t // w).double() + 0.5
    uvs = torch.full((B, S, Tq, h * w, 2), math.nan, device=DEV, dtype=torch.float64)
    codes = torch.full((B, S, Tq, h * w), -5, device=DEV, dtype=torch.int32)
    for b in range(B):
        use = torch.arange(S, device=DEV) if sel is None else sel[b].long()
        live = use >= 0
        pick = (lambda x: x[b]) if sel is None else (lambda x: x[use.clamp(min=0)])
        D, M, K = pool(pick(sd)), pick(sm).double(), pick(sk).double() / p
        z, R, Kt = pool(td[b]), tm[b].double(), tk[b].double() / p
        ray = torch.stack([(ux - Kt[:, 2:3]) / Kt[:, 0:1], (uy - Kt[:, 3:4]) / Kt[:, 1:2], torch.ones_like(z)], 1)
        X = R[:, :3, :3] @ (ray * z[:, None]) + R[:, :3, 3:]  # [Tq, 3, hw]
        Y = M[:, None, :3, :3].transpose(-1, -2) @ (X[None] - M[:, None, :3, 3:])  # [S, Tq, 3, hw]
        Z = Y[:, :, 2]
        u = (K[:, 0, None, None] * Y[:, :, 0] + K[:, 2, None, None] * Z) / Z
        v = (K[:, 1, None, None] * Y[:, :, 1] + K[:, 3, None, None] * Z) / Z
        known, front = (torch.isfinite(z) & (z > 0))[None].expand_as(Z), Z > 0
        on = known & front & (u >= 0) & (u < w) & (v >= 0) & (v < h)
        cell = torch.where(on, v.floor() * w + u.floor(), 0.0).long()
        seen = Z <= (1.0 + float(np.float32(EPS))) * torch.gather(D[:, None].expand(S, Tq, h * w), 2, cell)
        code = torch.where(seen, cell, -4)
        code = torch.where(on, code, -3)
        code = torch.where(known, torch.where(front, code, -2), -1).int()
        good = known & front & live[:, None, None]
        uvs[b] = torch.where(good[..., None], torch.stack([u, v], -1), math.nan)
        codes[b] = torch.where(live[:, None, None], code, torch.full_like(code, -5))
    return uvs.reshape(B, S, -1, 2), codes.reshape(B, S, -1)


def _turned(k, shift):
    """Keys [..., D] with the temporal pairs of the rotary embedding moved by `shift` frames, in double."""
    out = k.double().clone()
    phi = shift * torch.tensor([THETA ** (-i / ROPE_PAIRS) for i in range(ROPE_PAIRS)], device=DEV, dtype=torch.float64)
    x, y = out[..., 0:2 * ROPE_PAIRS:2].clone(), out[..., 1:2 * ROPE_PAIRS:2].clone()
    out[..., 0:2 * ROPE_PAIRS:2] = x * phi.cos() - y * phi.sin()
    out[..., 1:2 * ROPE_PAIRS:2] = x * phi.sin() + y * phi.cos()
    return out


def exact(case, seed):
    c, s = case, prepare(case, seed)
    if c["kind"] == "attn":
        return _exact_attention(s["q"], s["k"], s["v"], s["slot"], s["uv"], s["idx"], c["h"], c["w"], c["D"] ** -0.5)
    if c["kind"] == "retrieve":
        return _exact_retrieve(s, c["k"])
    if c["kind"] == "chunk":
        idx, score, count, sel = _exact_retrieve(s, c["k"])
        uv, code = _exact_reproject(s["tgt"], s["src"], c["h"], c["w"], c["p"], sel)
        return (idx, score, count, uv, code,
                *_exact_attention(s["q"], s["k"], s["v"], s["slot"], uv[0], code[0], c["h"], c["w"], c["D"] ** -0.5))
    if c["kind"] == "reproject":
        return _exact_reproject(s["tgt"], s["src"], c["h"], c["w"], c["p"])
    if c["kind"] == "rotation":
        # one centre: the depth cancels, so any depth does; a cell's own depth is not compared
        (tm, tk), (sm, sk) = s["tgt"], s["src"]
        ones = lambda m: torch.ones(*m.shape[:2], c["h"] * c["p"], c["w"] * c["p"], device=DEV)  # noqa: E731
        return _exact_reproject((ones(tm), tm, tk), (ones(sm), sm, sk), c["h"], c["w"], c["p"])[0], None
    if c["kind"] == "pack":
        T = F * c["h"] * c["w"]
        got = [x.double() for x in s["cache"]]
        for i, j in enumerate(s["sel"].tolist()):
            rows = slice((1 + i) * T, (2 + i) * T)
            got[0][:, rows], got[1][:, rows] = _turned(s["store"][0][:, j], F + i * F - F * j), s["store"][1][:, j].double()
        return tuple(got)
    # the anchor, the same place a ring ago, the two recent chunks and the chunk itself, at frames 0, F, 2F, 3F and 4F
    first, here = s["chunks"]
    h, w, p = c["h"], c["w"], c["p"]
    pooled = here[0].double().reshape(F, h, p, w, p).mean((-1, -3)).float()
    frames = (pooled, here[1], (here[2].double() / p).float())
    uv, code = _exact_reproject(tuple(x[None] for x in frames), tuple(x[None] for x in frames), h, w, 1)
    slot = _slots(5 * F, F)
    outs = []
    for n in range(c["layers"]):
        k = torch.cat([_turned(ch[4][n], F * part - 4 * F) for part, ch in enumerate([first] + [here] * 4)])
        v = torch.cat([ch[5][n] for ch in [first] + [here] * 4])
        outs.append(_exact_attention(here[3][n], k, v, slot, uv[0], code[0], h, w, c["D"] ** -0.5))
    return torch.stack([o for o, _ in outs]), torch.stack([l for _, l in outs])
