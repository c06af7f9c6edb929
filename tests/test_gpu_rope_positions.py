"""Rotary angles by position against the oracle: the most positions the table holds and one axis beyond (angles by token),
tiles with room for few positions, and sections that share their angles, do not, or are odd (by token)."""
import os
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import encoder_oracle as O
from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, dev_bf16, shared_weights

pytestmark = pytest.mark.gpu


def qkv_runs(enc, n_tokens, tile, positions):
    if not any(k.startswith("CS_") for k in os.environ):
        name = enc.cs_encoder_batch_kernel(B.STEPS["qkv"], n_tokens)
        assert name.startswith(f"gemm_kernel<{tile}> ") and name.endswith(f", {positions} positions"), name


# the most positions and one merge group beyond (by token): 64 x 64 and 64 x 128, 128 x 128 and 192 x 256 tiles hold all 128; 128 x 256
# have 6 KB left, 34 positions of 176 bytes; 256 x 256 with half tiles in the last round and 64-row tiles behind the full tile
# rows, which run the last item's rows from the 113th on
@pytest.mark.parametrize("sizes,tile,positions", [
    ([(28, 1792)], "64, 64, 2, 2, 6, 0", 128), ([(28, 1820)], "64, 128, 2, 4, 6, 0", 128),
    ([(28, 1792)] * 4, "128, 128, 4, 2, 6, 0", 128), ([(1792, 28)] * 9, "192, 256, 2, 4, 6, 0", 128),
    ([(476, 448)], "128, 256, 2, 4, 6, 0", 34), ([(504, 420)], "128, 256, 2, 4, 6, 0", 34),
    ([(1064, 1064), (28, 1792)], "256, 256, 2, 4, 6, 1", 128), ([(1064, 1064), (1820, 28)], "256, 256, 2, 4, 6, 1", 128)])
def test_positions(sizes, tile, positions):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"positions_{len(sizes)}_{sizes[-1][0]}_{sizes[-1][1]}", cfg, sizes, seq_len=4096, data_seed=sum(sizes[-1]))
    W = shared_weights("vit", w)
    qkv_runs(B.Encoder(cfg, W), int(w.cu_seqlens[-1]), tile, positions)
    check_items(f"images {sizes}", w, W, [len(sizes) - 1])


# the two-stage 128 x 128 tile, of which a CU holds two (a tower whose q and k columns are no whole 256-wide tiles)
@pytest.mark.parametrize("size,n", [((476, 56), 31), ((504, 56), 30)])
def test_positions_of_two_workgroups_a_cu(size, n):
    cfg = replace(wl.vit_7b_config(1), dtype="bf16", full_attn_layers=(), hidden=320, n_heads=4, mlp_dim=256, merger_hidden=256, out_hidden=256)
    w = wl.images_workload(f"pairs_{size[0]}", cfg, [size] * n, seq_len=2048, data_seed=n)
    # (scores large enough for the positions to matter: other axes move single elements by 0.18)
    W = {k: v * (8.0 if k.endswith("qkv.weight") else 1.0) for k, v in w.weights.items()}
    qkv_runs(B.Encoder(cfg, W), int(w.cu_seqlens[-1]), "128, 128, 2, 2, 6, 1", 34)
    check_items(f"{n} images {size}", w, W, [0, n - 1])


# (t, row, col) pairs: all of one size, three sizes, one axis alone, rows and clips alike, odd sizes
@pytest.mark.parametrize("sections", [(0, 16, 16), (6, 14, 12), (0, 0, 32), (12, 12, 8), (1, 16, 15)])
def test_sections(sections):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,), hidden=192, n_heads=3, head_dim=64, mlp_dim=512,
                  merger_hidden=256, out_hidden=256, rope_sections=sections)
    # (weights of the tiny widths large enough for the scores, and with them the positions, to matter)
    W = {n: np.clip(v, -16, 16) * (4.0 if "bias" not in n and v.ndim == 2 and n != "patch_embed.weight" else 1.0)
         for n, v in wl.images_workload(f"sections_{sections}", cfg, [(28, 28)], seq_len=512, data_seed=7).weights.items()}
    # an item of several time steps and a small one
    grid = np.array([[3, 8, 14], [2, 2, 6]], np.int32)
    n = grid.prod(1)
    x = wl.round_to_bf16(np.random.default_rng(3).standard_normal((int(n.sum()), cfg.patch_dim)).astype(np.float32))
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    out, _ = B.Encoder(cfg, W).cs_encode(dev_bf16(x), cu, grid)
    torch.cuda.synchronize()
    g, ref = out.double().cpu().numpy(), O.encode(cfg, W, x, cu, grid)
    moved = np.roll(sections, 1) if len(set(sections)) > 1 else sections   # other axes for the same pairs
    other = O.encode(replace(cfg, rope_sections=tuple(int(v) for v in moved)), W, x, cu, grid)
    rms = lambda d: np.sqrt((d ** 2).mean())
    print(f"sections {sections}: rms error {rms(g - ref):.3g}, with other axes {rms(other - ref):.3g}, of {rms(ref):.3g}", flush=True)
    assert rms(other - ref) > 20 * rms(g - ref)
    # bf16 operands (2^-9 each) through two layers whose scores, of a few units, turn them into as large errors of the weights
    assert rms(g - ref) < 0.015 * rms(ref)
