"""The measured work of this framework: encoder batches and their hand-off, through the public calls.

One pass is what the encoder executor and the consumer do for one packed batch: ``cs_encode`` (eager, or a
replayed graph) and ``cs_forward_embeddings`` into the consumer's input-embedding buffer; where the caller holds
decoded frames, ``cs_patchify`` in front of it.  An encoder is created once per tower and process, as a serving
process does, and batches of different inputs go through it; inputs, output rows, workspace and consumer buffer
belong to a state.

A case is a plain dict:

* ``tower``  "vit" (7B-style vision tower), "vit_video" (the same with rotary over t, row, col), "vit_tiny" (the
  small fp32 tower), "cls" (class-token tower, one item per 448 x 448 tile), "audio";
* ``items``  text, "HxW*count ..." in pixels for images, "FxHxW*count ..." for clips, "frames*count ..." for audio,
  "tiles" for the class-token tower;
* ``launch`` "eager" or "graph"; ``pixels`` start from fp32 frames instead of patch rows; ``chunk`` audio
  attention chunk in tokens (0: the whole clip); ``seq_len`` tokens per consumer sequence.
"""
from __future__ import annotations

import math
from dataclasses import replace

import numpy as np
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl

DEV = "cuda:0"
PATCH = wl.PATCH


def _case(name, tower, items, seq_len, launch="eager", pixels=False, chunk=0):
    c = {"tower": tower, "items": items, "seq_len": seq_len, "launch": launch, "pixels": pixels, "chunk": chunk}
    return dict(c, name=name) if name else c


def _sizes_text(sizes):
    return " ".join("x".join(str(v) for v in s) + "*1" for s in sizes)


def listed():
    return [
        # the tiny fp32 tower on one image: a call of a dozen short launches, latency alone
        _case("tiny_1x224", "vit_tiny", "224x224*1", 128),
        # the smallest request of the 7B-style tower: one thumbnail, weights and launches dominate
        _case("image_1x224", "vit", "224x224*1", 2048),
        # one ordinary image, replayed as a recorded graph (how a latency-bound server runs a fixed shape)
        _case("image_1x448_graph", "vit", "448x448*1", 2048, launch="graph"),
        # a handful of images of odd sizes from decoded frames: windows cut at the edges, ragged tiles everywhere
        _case("images_5_ragged_pixels", "vit", "84x140*1 252x476*1 56x56*1 700x420*1 364x644*1", 4096, pixels=True),
        # the benchmark's batch: eight 448 x 448 images
        _case("images_8x448", "vit", "448x448*8", 2048),
        # the largest: thirty-two images of mixed sizes in one variable-length batch
        _case("images_32_varlen", "vit", _sizes_text(wl.varlen_image_sizes()), 4096),
        # two 16-frame clips, full attention over 8192 patches
        _case("video_2x16x448", "vit_video", "16x448x448*2", 16384),
        # one 30 s clip, an utterance at a time
        _case("audio_1x30s", "audio", "3000*1", 2048),
        # sixteen 30 s clips, the batched transcription load
        _case("audio_16x30s", "audio", "3000*16", 2048),
        # clips of another length with block-diagonal (streaming-style) attention
        _case("audio_6_chunked", "audio", "1960*4 1208*2", 2048, chunk=100),
        # one tile of the class-token tower
        _case("tiles_1", "cls", "1", 2048),
        # eight tiles: an image of the tiling preprocessors, or several small ones
        _case("tiles_8", "cls", "8", 2048),
    ]


# The most a drawn case may cost: less than the largest listed one (110 940 patches, 154 TFLOP).
MAX_PATCHES, MAX_FRAMES, MAX_TILES = 90_000, 56_000, 96


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["images", "images", "images", "one_size", "video", "audio", "audio", "tiles"])
    if kind == "images":           # ragged images up to a total that is spread over the range
        total, sizes, n = _log_int(rng, 64, MAX_PATCHES), [], 0
        while len(sizes) < 48:
            h, w = rng.randint(2, 48), rng.randint(2, 48)
            if n + 4 * h * w > total:
                if sizes:
                    break
                h, w = max(2, int(math.sqrt(total) / 2 * rng.uniform(0.6, 1.0))), max(2, int(math.sqrt(total) / 2 * rng.uniform(0.6, 1.0)))
            sizes.append((28 * h, 28 * w))
            n += 4 * h * w
        return _case("", "vit", _sizes_text(sizes), 4096, pixels=rng.random() < 0.4)
    if kind == "one_size":         # a server that resizes to one shape
        h, w, n = 28 * rng.randint(4, 24), 28 * rng.randint(4, 24), _log_int(rng, 1, 24)
        return _case("", "vit", f"{h}x{w}*{n}", 2048, launch="graph" if n <= 4 else "eager", pixels=n > 4 and rng.random() < 0.5)
    if kind == "video":
        f, h, w = 2 * rng.randint(2, 12), 28 * rng.randint(4, 18), 28 * rng.randint(4, 18)
        per = f // 2 * (h // PATCH) * (w // PATCH)
        return _case("", "vit_video", f"{f}x{h}x{w}*{max(1, min(rng.randint(1, 4), 24_000 // per))}", 16384)
    if kind == "audio":
        frames, chunk = 8 * _log_int(rng, 8, 375), rng.choice([0, 0, 0, 52, 100])
        n = max(1, min(_log_int(rng, 1, 24), MAX_FRAMES // frames))
        return _case("", "audio", f"{frames}*{n}", 2048, chunk=chunk)
    return _case("", "cls", str(_log_int(rng, 1, MAX_TILES)), 2048)


# ---- what a serving process keeps: one encoder per tower -----------------------------------------------------
_weights, _encoders = {}, {}


def _config(case):
    if case["tower"] == "vit_tiny":
        return wl.vit_tiny_config()
    if case["tower"] in ("vit", "vit_video"):
        return wl.vit_7b_config(out_dtype="bf16", rope_sections=(0, 20, 20) if case["tower"] == "vit" else (8, 16, 16))
    if case["tower"] == "cls":
        return wl.vit_cls_config(out_dtype="bf16")
    return replace(wl.audio_config(out_dtype="bf16"), attn_chunk=case["chunk"])


def _tower_weights(cfg):
    """Random-init weights of workloads.make_weights' distributions, drawn on the GPU (a tower has 0.3 - 0.7 G of them)."""
    key = (cfg.arch, cfg.hidden)
    if key not in _weights:
        gen = torch.Generator(device=DEV)
        gen.manual_seed(0)
        W = {}
        for name, shape, kind in wl.weight_shapes(cfg):
            a = torch.randn(shape, generator=gen, device=DEV) * 0.02
            if kind == "g":
                a += 1.0
            if kind == "s":
                a += 0.1
            if kind == "kb":
                a[cfg.hidden:2 * cfg.hidden] = 0.0
            if cfg.dtype == "bf16":
                a = a.bfloat16().float()
            W[name] = a.cpu().numpy()
        _weights[key] = W
    return _weights[key]


def _encoder(cfg):
    if cfg not in _encoders:
        _encoders[cfg] = B.Encoder(cfg, _tower_weights(cfg))
    return _encoders[cfg]


# ---- batches --------------------------------------------------------------------------------------------------
def _items(case):
    """[(shape in the case's own units), ...], one entry per item."""
    if case["tower"] == "cls":
        return [(448, 448)] * int(case["items"])
    out = []
    for part in case["items"].split():
        dims, n = part.split("*")
        out += [tuple(int(v) for v in dims.split("x"))] * int(n)
    return out


def _grid(case, cfg):
    """grid_thw of the batch, as cs_encode takes it."""
    g = []
    for it in _items(case):
        if case["tower"] == "audio":
            g.append((1, 1, it[0]))
        elif len(it) == 3:
            g.append((it[0] // cfg.temporal_patch, it[1] // PATCH, it[2] // PATCH))
        else:
            g.append((1, it[0] // PATCH, it[1] // PATCH))
    return np.asarray(g, np.int32)


def _out_rows(case, cfg, grid):
    n = grid.astype(np.int64).prod(1)
    return n // (2 * cfg.merge) if case["tower"] == "audio" else n // (cfg.merge * cfg.merge)


class _State:
    pass


def prepare(case, seed):
    cfg = _config(case)
    s = _State()
    s.enc, s.cfg, s.pixels = _encoder(cfg), cfg, case["pixels"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    in_dtype = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    s.grid = _grid(case, cfg)
    n = s.grid.astype(np.int64).prod(1)
    s.cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    N, tp = int(s.cu[-1]), cfg.temporal_patch
    if case["tower"] == "audio":                                      # log-mel frames, N(0, 1)
        s.x = torch.randn(N, cfg.patch_dim, generator=gen, device=DEV).to(in_dtype)
    elif s.pixels:                                                    # decoded stills, fp32, U(0, 1)
        s.dims = [(1, h, w) for h, w in _items(case)]
        s.frames = torch.rand(sum(3 * h * w for _, h, w in s.dims), generator=gen, device=DEV)
    elif len(_items(case)[0]) == 3:                                   # clips: every frame its own pixels
        s.x = torch.rand(N, cfg.patch_dim, generator=gen, device=DEV).to(in_dtype)
    else:                                                             # stills: shown tp times
        px = torch.rand(N, 3, 1, PATCH * PATCH, generator=gen, device=DEV).to(in_dtype)
        s.x = px.expand(N, 3, tp, PATCH * PATCH).reshape(N, cfg.patch_dim).contiguous()
        del px
    n_out, ws_bytes = s.enc.cs_encoder_query(s.cu, s.grid)
    out_dtype = torch.bfloat16 if cfg.out_dtype == "bf16" else torch.float32
    s.out = torch.empty(n_out, cfg.out_hidden, dtype=out_dtype, device=DEV)
    s.workspace = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
    # the consumer: one sequence per item holding its text-token embeddings, and a span of placeholders at a place of its own
    rows, seq_len = _out_rows(case, cfg, s.grid), int(case["seq_len"])
    s.dst = (torch.randn(len(rows) * seq_len, cfg.out_hidden, generator=gen, device=DEV, dtype=out_dtype)).mul_(0.02)
    rng = np.random.default_rng(int(seed))
    idx = [b * seq_len + int(rng.integers(0, seq_len - int(m) + 1)) + np.arange(int(m), dtype=np.int64) for b, m in enumerate(rows)]
    s.idx = torch.from_numpy(np.concatenate(idx)).to(DEV)
    s.graph = None
    if case["launch"] == "graph":
        torch.cuda.synchronize()
        s.graph = s.enc.cs_encode_graph_create(s.x, s.cu, s.grid, s.out, s.workspace, torch.cuda.Stream())
    return s


def run(state):
    s = state
    if s.graph is not None:
        s.graph.cs_encode_graph_launch()
    elif s.pixels:
        x, cu, grid = B.cs_patchify(s.frames, s.dims, s.cfg.temporal_patch)
        s.enc.cs_encode(x, cu, grid, out=s.out, workspace=s.workspace)
    else:
        s.enc.cs_encode(s.x, s.cu, s.grid, out=s.out, workspace=s.workspace)
    B.cs_forward_embeddings(s.out, s.idx, s.dst)
    return {"embeddings": s.out, "sequences": s.dst}


def work(case):
    """Bytes: pixels or patch rows, weights, index read once; embedding rows written, read and placed.  Flops: the matrix products and attention the method has, no padding, no masked-out scores."""
    cfg = _config(case)
    grid = _grid(case, cfg)
    n_item = grid.astype(np.int64).prod(1)
    N, D, I, L = int(n_item.sum()), cfg.hidden, cfg.mlp_dim, cfg.n_layers
    rows = int(_out_rows(case, cfg, grid).sum())
    es_in, es_out = (2 if cfg.dtype == "bf16" else 4), (2 if cfg.out_dtype == "bf16" else 4)
    w_elems = sum(int(np.prod(shape)) for _, shape, _ in wl.weight_shapes(cfg))
    in_bytes = 4 * sum(3 * h * w for h, w in _items(case)) if case["pixels"] else N * cfg.patch_dim * es_in
    nbytes = in_bytes + w_elems * es_in + rows * (3 * cfg.out_hidden * es_out + 8)
    f = 0
    if cfg.arch == "audio":
        tok = n_item // 2
        f += 2 * N * 3 * cfg.patch_dim * D + 2 * (N // 2) * 3 * D * D + 2 * rows * D * cfg.out_hidden
        att = sum((int(t) // case["chunk"]) * case["chunk"] ** 2 + (int(t) % case["chunk"]) ** 2 if case["chunk"] else int(t) ** 2 for t in tok)
        N, att, mlp = N // 2, 4 * att * D * L, 2 * D * I
    else:
        f += 2 * N * cfg.patch_dim * D + 2 * rows * (4 * D * cfg.merger_hidden + cfg.merger_hidden * cfg.out_hidden)
        if cfg.arch == "vit_cls":
            tok = n_item + 1
            N, att, mlp = int(tok.sum()), 4 * int((tok ** 2).sum()) * D * L, 2 * D * I
        else:
            def cuts(v):
                return [cfg.window] * (v // cfg.window) + ([v % cfg.window] if v % cfg.window else []) if cfg.window > 0 else [v]
            win = sum(int(t) * sum((a * b) ** 2 for a in cuts(int(h)) for b in cuts(int(w))) for t, h, w in grid)
            full = int((n_item ** 2).sum())
            n_full = len(cfg.full_attn_layers) if cfg.window > 0 else L
            att, mlp = 4 * D * (win * (L - n_full) + full * n_full), 3 * D * I
    f += att + L * N * (2 * 4 * D * D + 2 * mlp)
    return {"bytes": float(nbytes), "flops": float(f)}


def tolerance(case):
    """An item run alone and inside a batch takes other tiles and other orders of its fp32 sums over the same bf16
    products: two correct evaluations.  Measured between the two, on the bf16 rows: vision tower rel 0.0045, max
    0.022; audio 0.0043, 0.022; class-token tower 0.0032, 0.014.  Four times the largest."""
    return {"rel": 0.018, "max": 0.09}
