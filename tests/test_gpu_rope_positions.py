"""Rotary angles by position against the oracle: the most positions the table holds and one axis beyond (angles by token),
tiles with room for few positions, and sections that share their angles, do not, or are odd (by token)."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import encoder_oracle as O
from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, dev_bf16, shared_weights

pytestmark = pytest.mark.gpu


# 128 positions; 130; 128 x 256 tiles with 7 KB left: 40 positions of 176 bytes fill it, 42 do not; 256 x 256 tiles with a light tail
@pytest.mark.parametrize("sizes", [[(28, 1792)], [(28, 1820)], [(560, 420)], [(588, 420)], [(28, 1792), (1064, 1064)], [(1820, 28), (1064, 1064)]])
def test_positions(sizes):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"positions_{sizes[0][0]}_{sizes[0][1]}", cfg, sizes, seq_len=4096, data_seed=sum(sizes[0]))
    check_items(f"images {sizes}", w, shared_weights("vit", w), [0])


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
