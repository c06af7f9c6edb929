"""The two ways an attention tile is addressed: tiles inside the batch by a scalar base and kept offsets, the batch's last
tile (whose rows beyond the end must not be read) and far pitches of v^T by full addresses."""
import math

import numpy as np
import pytest
import torch

from oracle import encoder_oracle as O
from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import dev_bf16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def attend(segs, nh, dh, pitch):
    n = sum(segs)
    rng = np.random.default_rng(n + dh)
    q = wl.round_to_bf16(rng.standard_normal((n, nh * dh), dtype=np.float32) * np.float32(1.4426950408889634 / math.sqrt(dh)))
    k, v = (wl.round_to_bf16(rng.standard_normal((n, nh * dh), dtype=np.float32)) for _ in range(2))
    item = np.repeat(np.arange(len(segs)), segs)
    q64 = q.astype(np.float64) * math.sqrt(dh) * math.log(2.0)
    ref = O.attention(q64.reshape(n, nh, dh), k.reshape(n, nh, dh).astype(np.float64), v.reshape(n, nh, dh).astype(np.float64),
                      item[:, None] == item[None, :]).reshape(n, nh * dh)
    vt = torch.empty(nh * dh, pitch, device=DEV, dtype=torch.bfloat16)
    vt[:, :(n + 63) // 64 * 64] = float("nan")                         # nothing behind the batch may reach a result
    vt[:, :n] = dev_bf16(np.ascontiguousarray(v.T))
    rows = torch.full((n + 64, 2 * nh * dh), float("nan"), device=DEV, dtype=torch.bfloat16)
    rows[:n] = dev_bf16(np.concatenate([q, k], 1))
    out = torch.full((n, nh * dh), 7.0, device=DEV, dtype=torch.bfloat16)
    B.cs_attention_varlen(rows, vt, out, np.concatenate([[0], np.cumsum(segs)]), nh, dh)
    torch.cuda.synchronize()
    return np.abs(out.double().cpu().numpy() - ref).max()


# one segment or two, ending one group of four before, at and behind a tile's end: windows of one tile (all segments <= 64)
# and the 256-query kernels
@pytest.mark.parametrize("dh", [64, 80])
@pytest.mark.parametrize("segs", [[4], [60], [64], [60, 64], [64, 4], [68], [124], [128], [132], [128, 68], [260, 256], [316, 4]])
def test_tile_ends(dh, segs):
    # probabilities and outputs are rounded to bf16 (2^-9 relative), |v| up to ~4
    assert attend(segs, 2, dh, (sum(segs) + 63) // 64 * 64) <= 2e-2


# the pitch up to which 32-bit offsets reach (rows of the head and one step of a 512-thread workgroup), and the next one;
# 1.4 GB (head dimension 64) and 1.5 GB (80) of v^T, of which the columns of the batch are touched
@pytest.mark.parametrize("dh", [64, 80])
@pytest.mark.parametrize("beyond", [False, True])
def test_far_pitch(dh, beyond):
    pitch = 0x7fffffff // (2 * (dh + 32)) // 4 * 4
    assert attend([260, 132], 1, dh, pitch + 4 * beyond) <= 2e-2
