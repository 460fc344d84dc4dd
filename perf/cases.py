"""The calls whose time matters, as a program that compresses visual tokens makes them.

Every case is a problem size, an element type and an entry point: the whole pass
(``ttf_compress``), a stream segment against a rolling anchor (``ttf_compress_segment``), the
tied batch (``ttf_compress_tied``), the rebuilt layout (``ttf_restore_map`` + ``ttf_restore``)
and the adaptive threshold (``ttf_select_threshold`` + ``ttf_regate``).  ``listed`` holds the
shapes the repository's own configurations name and the ones next to them; ``draw`` gives
others from the ranges they stand for.

Inputs are drawn on the GPU with the recipe of ``workloads/ttf_gen.py`` ("anchored"): a latent
scene, one low-noise frame per scene, every other frame the scene moved by at most the radius,
with noise of a per-token amplitude and 10 % of the cells replaced.  As there, tokens whose
similarity would lie within 2e-3 of the threshold are drawn again, so that two correct
implementations keep the same rows.
"""
import math

import torch

import paper_2605_07355_amd as ttf

CLEAN = 0.3          # noise of the low-noise frame of a scene
SIGMA = 0.628        # noise scale of the others: amplitude uniform in [0, 2 SIGMA)
P_CHANGE = 0.10      # share of cells replaced by fresh content
SCENE = 32           # frames per scene of clips of more than 64 frames (shorter ones are one scene)
FUSED = 0.67         # requested fused fraction of the adaptive threshold

DRAWN = 1 << 30      # most input bytes of a drawn case (the largest listed ones have twice that)


def _case(name, path, B, F, H, W, C, dtype, r, t):
    return {"name": name, "path": path, "B": B, "F": F, "H": H, "W": W, "C": C, "dtype": dtype, "r": r, "t": t}


def listed():
    return [
        # the smallest call: a thumbnail clip in fp32, bound by latency and launches
        _case("clip_tiny", "compress", 1, 4, 8, 8, 256, "f32", 1, 0.70),
        # one clip of a small model, as an interactive request brings it
        _case("clip_2b", "compress", 1, 32, 16, 16, 2048, "bf16", 1, 0.70),
        # a full batch of clips of a large model: the headline configuration
        _case("batch_8b", "compress", 16, 32, 16, 16, 4096, "bf16", 1, 0.70),
        # long videos with scene cuts: few clips, many frames, most rows kept
        _case("long_video", "compress", 2, 256, 16, 16, 4096, "bf16", 1, 0.70),
        # high-resolution grids with the wide 5x5 window
        _case("highres_wide", "compress", 4, 64, 32, 32, 4096, "bf16", 2, 0.70),
        # the full batch in fp32 features
        _case("batch_fp32", "compress", 16, 32, 16, 16, 4096, "f32", 1, 0.70),
        # a grid that is no multiple of the tile
        _case("odd_grid", "compress", 16, 32, 14, 14, 4096, "bf16", 1, 0.70),
        # odd in every size: grid, frame count, and channels that are not whole 32-channel steps
        _case("odd_channels", "compress", 3, 23, 24, 18, 1000, "bf16", 1, 0.70),
        # one short segment of a live stream against the rolling anchor frame
        _case("stream_segment", "segment", 1, 8, 16, 16, 4096, "bf16", 1, 0.70),
        # four views of one scene under the tied-batch rule
        _case("tied_views", "tied", 4, 32, 16, 16, 4096, "bf16", 1, 0.70),
        # the full layout rebuilt from compressed rows
        _case("restore", "restore", 8, 32, 16, 16, 4096, "bf16", 1, 0.70),
        # threshold picked per clip from stored similarities, gate and rows redone with it
        _case("adaptive", "adaptive", 8, 32, 16, 16, 4096, "bf16", 1, 0.70),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["compress"] * 6 + ["segment", "tied", "restore", "adaptive"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    step = rng.choice([256, 128, 32, 8])                   # whole K-steps more often than not
    C = max(256, min(4096, _log(rng, 256, 4096) // step * step))
    H = rng.choice([16, 32, rng.randint(8, 32)])
    W = rng.choice([16, 32, rng.randint(8, 32)])
    F = _log(rng, 4, 256)
    B = _log(rng, 2 if path == "tied" else 1, 16)
    row = H * W * C * (2 if dtype == "bf16" else 4)
    F = max(4, min(F, DRAWN // row))
    B = max(1, min(B, DRAWN // (row * F)))
    return {"path": path, "B": B, "F": F, "H": H, "W": W, "C": C, "dtype": dtype, "r": rng.choice([0, 1, 1, 1, 2]),
            "t": rng.choice([0.60, 0.70, 0.70, 0.80])}


def _scene(case):
    return SCENE if case["F"] > 64 else case["F"]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _frames(case, seed, shared_motion=False):
    """[B,F,H,W,C] features and, for every clip, the low-noise frame of its first scene."""
    B, F, H, W, C, r, t = (case[k] for k in ("B", "F", "H", "W", "C", "r", "t"))
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = _gen(seed)
    rnd = dict(device="cuda", generator=g)
    x = torch.empty((B, F, H, W, C), dtype=dtype, device="cuda")
    first_clean = None
    M = 1 if shared_motion else B                          # independent motion fields, amplitudes and masks
    yy = torch.arange(H, device="cuda")[None, :, None]
    xx = torch.arange(W, device="cuda")[None, None, :]
    clip = torch.arange(B, device="cuda")[:, None, None]
    scene = _scene(case)
    for k0 in range(0, F, scene):
        k1 = min(F, k0 + scene)
        latent = torch.randn((B, H, W, C), **rnd)
        clean = (latent + CLEAN * torch.randn((B, H, W, C), **rnd)).to(dtype)
        cinv = clean.float().norm(dim=-1)
        kstar = torch.randint(k0, k1, (M,), **rnd).expand(B)
        first_clean = clean if first_clean is None else first_clean
        for k in range(k0, k1):
            # motion, constant on 4x4 regions
            off = torch.randint(-r, r + 1, (2, M, -(-H // 4), -(-W // 4)), **rnd)
            off = off.repeat_interleave(4, 2).repeat_interleave(4, 3)[:, :, :H, :W].expand(2, B, H, W)
            ys, xs = (yy - off[0]).clamp(0, H - 1), (xx - off[1]).clamp(0, W - 1)
            amp = 2 * SIGMA * torch.rand((M, H, W), **rnd).expand(B, H, W)
            base = latent[clip, ys, xs]
            f = (base + amp[..., None] * torch.randn((B, H, W, C), **rnd)).to(dtype)
            c = clean[clip, ys, xs]
            s = (f.float() * c.float()).sum(-1) / (f.float().norm(dim=-1) * cinv[clip, ys, xs])
            # too close to the threshold to be sure of: drawn again, without noise
            f = torch.where(((s - t).abs() < 2e-3)[..., None], base.to(dtype), f)
            fresh = torch.rand((M, H, W), **rnd).expand(B, H, W) < P_CHANGE
            f = torch.where(fresh[..., None], torch.randn((B, H, W, C), **rnd).to(dtype), f)
            x[:, k] = torch.where((kstar == k)[:, None, None, None], clean, f)
    return x, first_clean


def _buffers(case, dtype):
    b = ttf.TTFBuffers.allocate(case["B"], case["F"], case["H"], case["W"], case["C"], dtype, torch.device("cuda"))
    for v in (b.tokens_out, b.pos_ids, b.src_index):       # rows past the last one are left as they are
        v.zero_()
    return b


def prepare(case, seed):
    B, F, H, W, C, r, t = (case[k] for k in ("B", "F", "H", "W", "C", "r", "t"))
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    s = {"case": case}
    path = case["path"]
    if path == "tied":
        s["x"] = _frames(case, seed, shared_motion=True)[0]
        s["buf"] = ttf.TTFTiedBuffers.allocate(B, F, H, W, C, dtype, torch.device("cuda"), r=r)
        for v in (s["buf"].tokens_out, s["buf"].pos_ids, s["buf"].src_index):
            v.zero_()
        return s
    if path == "adaptive":
        # stored matches of an earlier pass: two modes of similarity, cells within the window
        g = _gen(seed)
        rnd = dict(device="cuda", generator=g)
        s["x"] = torch.randn((B, F, H, W, C), **rnd).to(dtype)
        b = s["buf"] = _buffers(case, dtype)
        hi = 0.90 + 0.04 * torch.randn((B, F, H * W), **rnd)
        lo = 0.35 + 0.15 * torch.randn((B, F, H * W), **rnd)
        b.best_sim.copy_(torch.where(torch.rand((B, F, H * W), **rnd) < FUSED, hi, lo).clamp(-1, 1))
        i = torch.arange(H * W, device="cuda")
        off = torch.randint(-r, r + 1, (2, B, F, H * W), **rnd)
        b.best_idx.copy_((i // W + off[0]).clamp(0, H - 1) * W + (i % W + off[1]).clamp(0, W - 1))
        b.anchor_index.copy_(torch.randint(0, F, (B,), **rnd))
        at = (torch.arange(B, device="cuda"), b.anchor_index.long())
        b.best_sim[at] = 1.0
        b.best_idx[at] = i.int()
        s["out"] = ttf.TTFOutput(b, B, F, H, W, C)
        s["thresholds"] = torch.empty((B,), dtype=torch.float32, device="cuda")
        return s
    s["x"], clean = _frames(case, seed)
    s["buf"] = _buffers(case, dtype)
    if path == "segment":
        s["anchor"] = clean                                # the frame that closed the previous segment
    if path == "restore":
        s["out"] = ttf.ttf_compress(s["x"], r=r, t=t, buffers=s["buf"])
        s["rows"] = s["out"].total_rows
        s["map"] = torch.empty((B, F, H * W), dtype=torch.int32, device="cuda")
        s["full"] = torch.empty_like(s["x"])
    return s


def _outputs(b, *names):
    return {n: getattr(b, n) for n in names}


_PASS = ("tokens_out", "pos_ids", "src_index", "row_offsets", "kept_count", "anchor_index", "fuse_map", "best_sim",
         "best_idx")


def run(s):
    case, path = s["case"], s["case"]["path"]
    if path == "compress":
        return _outputs(ttf.ttf_compress(s["x"], r=case["r"], t=case["t"], buffers=s["buf"]).buffers, *_PASS)
    if path == "segment":
        out = ttf.ttf_compress_segment(s["x"], s["anchor"], frame_offset=64, r=case["r"], t=case["t"], buffers=s["buf"])
        return _outputs(out.buffers, *_PASS)
    if path == "tied":
        b = ttf.ttf_compress_tied(s["x"], r=case["r"], t=case["t"], buffers=s["buf"])
        return _outputs(b, "tokens_out", "pos_ids", "src_index", "kept_count", "anchor_index", "fuse_map", "best_sim",
                        "best_idx", "mean_sim")
    if path == "restore":
        rmap = ttf.ttf_restore_map(s["out"], s["map"])
        full = ttf.ttf_restore(s["buf"].tokens_out, s["rows"], rmap, case["H"], case["W"], s["full"])
        return {"map": rmap, "full": full}
    thr = ttf.ttf_select_threshold(s["out"], FUSED, s["thresholds"])
    out = ttf.ttf_regate(s["x"], s["out"], thr)
    return {"thresholds": thr, **_outputs(out.buffers, "tokens_out", "pos_ids", "src_index", "row_offsets",
                                          "kept_count", "fuse_map")}


def _fused_share(case):
    """Expected share of source tokens that fuse, from the recipe's closed form."""
    if case["path"] == "adaptive":
        return FUSED
    amp = math.sqrt(max(0.0, 1 / ((1 + CLEAN ** 2) * case["t"] ** 2) - 1))
    share = (1 - P_CHANGE) * min(1.0, amp / (2 * SIGMA))
    if case["path"] == "tied":                             # every view has to agree, but they share their amplitudes
        share *= 0.97
    return share * _scene(case) / case["F"]             # only the anchor's own scene fuses


def work(case):
    B, F, H, W, C, r = (case[k] for k in ("B", "F", "H", "W", "C", "r"))
    row = C * (2 if case["dtype"] == "bf16" else 4)
    tokens, frame = B * F * H * W, B * H * W
    source = tokens if case["path"] == "segment" else tokens - frame
    kept = source * (1 - _fused_share(case)) + (0 if case["path"] == "segment" else frame)
    search = source * (2.0 * (2 * r + 1) ** 2 + 2.0) * C
    ids = 16                                               # position triple and flat index of a row
    if case["path"] == "restore":
        return {"bytes": kept * row + tokens * (row + 8) + 4 * kept, "flops": 0}
    if case["path"] == "adaptive":                         # similarities, cells and the kept rows
        return {"bytes": tokens * 12 + kept * (2 * row + ids), "flops": 0}
    each = 12 if case["path"] != "tied" else 4             # fuse_map, best_sim, best_idx of every token
    anchor = frame * row if case["path"] == "segment" else 0
    return {"bytes": tokens * (row + each) + anchor + kept * (row + ids), "flops": search}


def tolerance(case):
    if case["path"] in ("restore", "adaptive"):
        return "exact"                                     # copies, integers and an exact order statistic
    # similarities: fp32 sums of C terms, or fp32 values in 24-bit pieces.  Of the whole numbers only
    # the best cell of a replaced token, whose candidates can tie within rounding, may differ.
    return {"rel": 2e-6, "max": 1e-5, "differ": 1e-3}


def _window_exact(x, anchor, r):
    """Cosines of the frame x with every in-grid cell of its window of the anchor frame, [B,K,H,W] in fp64."""
    B, H, W, C = x.shape
    xd, ad = x.double(), anchor.double()
    xn, an = xd.norm(dim=-1), ad.norm(dim=-1)
    win = torch.full((B, (2 * r + 1) ** 2, H, W), -math.inf, dtype=torch.float64, device=x.device)
    for slot in range(win.shape[1]):
        dy, dx = slot // (2 * r + 1) - r, slot % (2 * r + 1) - r
        ys, xs = slice(max(0, -dy), min(H, H - dy)), slice(max(0, -dx), min(W, W - dx))
        ya, xa = slice(max(0, dy), min(H, H + dy)), slice(max(0, dx), min(W, W + dx))
        dot = torch.zeros_like(xn[:, ys, xs])
        for c in range(0, C, 512):
            dot += (xd[:, ys, xs, c:c + 512] * ad[:, ya, xa, c:c + 512]).sum(-1)
        win[:, slot, ys, xs] = dot / (xn[:, ys, xs] * an[:, ya, xa])
    return win


def exact(case, seed):
    """The similarities in 64 bits; everything else of the outputs is copies and whole numbers."""
    path, r = case["path"], case["r"]
    if path in ("restore", "adaptive"):
        return None
    x, clean = _frames(case, seed, shared_motion=path == "tied")
    B, F = x.shape[:2]
    clip = torch.arange(B, device="cuda")
    if path == "segment":
        a, frame = None, clean
    else:
        sums = torch.stack([x[:, k].double().sum((1, 2)) for k in range(F)], 1)
        score = torch.nn.functional.cosine_similarity(sums, sums.sum(1, keepdim=True), dim=-1)
        a = score.mean(0).argmax().expand(B) if path == "tied" else score.argmax(1)
        frame = x[clip, a]
    best, mean = [], []
    for k in range(F):
        win = _window_exact(x[:, k], frame, r)
        if path == "tied":                                 # one cell for all views: the best in the mean
            m, slot = win.mean(0, keepdim=True).max(1)
            mean.append(m[0])
            best.append(win.gather(1, slot[:, None].expand(B, 1, *slot.shape[1:]))[:, 0])
        else:
            best.append(win.amax(1))
        if a is not None:
            best[-1] = torch.where((a == k)[:, None, None], 1.0, best[-1])
            if path == "tied":
                mean[-1] = torch.where(a[0] == k, 1.0, mean[-1])
    want = dict.fromkeys(_PASS if path != "tied" else ("tokens_out", "pos_ids", "src_index", "kept_count", "anchor_index",
                                                       "fuse_map", "best_sim", "best_idx", "mean_sim"))
    want["best_sim"] = torch.stack(best, 1).flatten(2)
    if path == "tied":
        want["mean_sim"] = torch.stack(mean, 0).flatten(1)
    return want
