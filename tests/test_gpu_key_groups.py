"""The attention kernels whose waves share out the key tiles of an item, on their own and in a batch of unequal clips:
groups without a tile, groups whose maxima lie far apart, ragged segments."""
import math
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import encoder_oracle as O
from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import MAX_ABS, MIN_COS, dev_bf16, shared_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def attend(segs, nh, q, k, v, groups):
    """q as the kernel takes it (scale and log2 e folded in); (rows of the kernel, rows of the oracle)"""
    dh, n = 64, sum(segs)
    cu = np.concatenate([[0], np.cumsum(segs)])
    item = np.repeat(np.arange(len(segs)), segs)
    q64 = q.astype(np.float64) * math.sqrt(dh) * math.log(2.0)
    ref = O.attention(q64.reshape(n, nh, dh), k.reshape(n, nh, dh).astype(np.float64), v.reshape(n, nh, dh).astype(np.float64),
                      item[:, None] == item[None, :]).reshape(n, nh * dh)
    vt = torch.zeros(nh * dh, (n + 7) // 8 * 8, device=DEV, dtype=torch.bfloat16)
    vt[:, :n] = dev_bf16(np.ascontiguousarray(v.T))
    out = torch.full((n, nh * dh), 7.0, device=DEV, dtype=torch.bfloat16)
    B.cs_attention_varlen_groups(dev_bf16(np.concatenate([q, k], 1)), vt, out, cu, nh, dh, groups)
    torch.cuda.synchronize()
    return out.double().cpu().numpy(), ref


# sharp > 1: queries scaled up, so that scores differ by dozens; order: keys growing or shrinking along a segment, which
# moves the largest scores to its end or its start, or large in every other tile, which parts the groups' maxima
@pytest.mark.parametrize("groups", [1, 2, 4])
@pytest.mark.parametrize("segs", [[1500, 32], [64, 1028], [580, 4], [4], [64], [68, 132, 196, 260], [1024, 128]])
@pytest.mark.parametrize("sharp,order", [(1.0, "even"), (6.0, "up"), (6.0, "down"), (6.0, "tiles")])
def test_groups_match_oracle(groups, segs, sharp, order):
    rng = np.random.default_rng(len(segs) + sum(segs))
    nh, n = 2, sum(segs)
    q = wl.round_to_bf16(rng.standard_normal((n, nh * 64), dtype=np.float32) * np.float32(sharp * 1.4426950408889634 / 8))
    k = rng.standard_normal((n, nh * 64), dtype=np.float32)
    at = np.arange(n, dtype=np.float32)
    k *= {"even": 1 + 0 * at, "up": 1 + at / n, "down": 2 - at / n, "tiles": 0.25 + 1.5 * (at // 64 % 2)}[order][:, None]
    k, v = wl.round_to_bf16(k), wl.round_to_bf16(rng.standard_normal((n, nh * 64), dtype=np.float32))
    got, ref = attend(segs, nh, q, k, v, groups)
    # probabilities and outputs are rounded to bf16 (2^-9 relative), |v| up to ~4: the bound of the kernel without groups
    assert np.abs(got - ref).max() <= 2e-2


@pytest.mark.parametrize("frames", [[2600, 64], [8, 1208, 72]])
def test_audio_clips_of_unequal_length(frames):
    cfg = replace(wl.audio_config(2), attn_chunk=0)
    clips = [wl.audio_workload(f"clip{f}", cfg, 1, f, seq_len=2048, data_seed=f) for f in frames]
    W = shared_weights("audio", clips[0])
    cu = np.concatenate([[0], np.cumsum(frames)]).astype(np.int32)
    grid = np.asarray([(1, 1, f) for f in frames], np.int32)
    assert B.cs_plan_attention(cfg, cu, grid)[0].key_groups == 2
    enc = B.Encoder(cfg, W)
    out, _ = enc.cs_encode(dev_bf16(np.concatenate([c.patches for c in clips])), cu, grid)
    torch.cuda.synchronize()
    got, row = out.double().cpu().numpy(), 0
    for c in clips:
        ref = O.encode(cfg, W, c.patches, c.cu_seqlens, c.grid_thw)
        g = got[row:row + len(ref)]
        row += len(ref)
        cos = (g * ref).sum(1) / (np.linalg.norm(g, axis=1) * np.linalg.norm(ref, axis=1))
        assert np.abs(g - ref).max() <= MAX_ABS and cos.min() >= MIN_COS, (c.name, np.abs(g - ref).max(), cos.min())
    assert row == len(got)


# the keys from 64 on to 127 (the first tile of the second group), or all from 64 on to the last 64, score -inf for every
# query: they weigh nothing, in whichever group they fall
@pytest.mark.parametrize("groups", [1, 2, 4])
@pytest.mark.parametrize("n,lo,hi", [(128, 64, 128), (300, 64, 128), (1028, 64, 128), (1028, 64, 964), (640, 64, 640)])
def test_tiles_of_keys_without_weight(groups, n, lo, hi):
    rng = np.random.default_rng(n + lo)
    q = wl.round_to_bf16(rng.standard_normal((n, 64), dtype=np.float32) * np.float32(1.4426950408889634 / 8))
    k = wl.round_to_bf16(rng.standard_normal((n, 64), dtype=np.float32))
    v = wl.round_to_bf16(rng.standard_normal((n, 64), dtype=np.float32))
    q[:, 0], k[:, 0] = 2.0 ** 70, 0.0
    k[lo:hi, 0] = -(2.0 ** 70)                 # products of -2^140: beyond fp32
    got, ref = attend([n], 1, q, k, v, groups)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 2e-2     # as above
