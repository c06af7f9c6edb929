"""Full attention of few queries runs its 256-query items, and the short last ones, as workgroups of 64 queries: batches on
both sides of that rule, items of one block and of several, last blocks of every length."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, dev_bf16, shared_weights

pytestmark = pytest.mark.gpu


# 16 heads: 32 blocks of 64 queries make 512 workgroups (2048 tokens; 25 and 7 blocks), 2052 tokens one block more; the
# others are below, with last blocks of 4, 24, 32, 36 and 64 queries, some of them short items behind a 256-query one
@pytest.mark.parametrize("sizes,queries", [([(896, 448)], 64), ([(560, 560), (224, 364)], 64), ([(532, 756)], 256), ([(532, 532), (224, 308)], 64),
                                           ([(28, 28)], 64), ([(28, 28), (252, 476), (56, 84)], 64),
                                           ([(112, 112), (224, 252), (140, 364)], 64)])
def test_images(sizes, queries):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(0, 1))
    w = wl.images_workload(f"blocks_{len(sizes)}", cfg, sizes, seq_len=8192, data_seed=sum(h + v for h, v in sizes))
    assert B.cs_plan_attention_queries(cfg, w.cu_seqlens, w.grid_thw) == queries
    check_items(f"images {sizes}", w, shared_weights("vit", w), range(len(sizes)))


@pytest.mark.parametrize("frames,queries", [([8], 64), ([512, 136], 64), ([1000, 8, 264], 64), ([1016] * 4, 256)])
def test_clips(frames, queries):
    cfg = wl.audio_config(2)
    clips = [wl.audio_workload(f"clip{f}", cfg, 1, f, seq_len=2048, data_seed=f) for f in frames]
    enc = B.Encoder(cfg, shared_weights("audio", clips[0]))
    cu = np.concatenate([[0], np.cumsum(frames)]).astype(np.int32)
    grid = np.asarray([(1, 1, f) for f in frames], np.int32)
    assert B.cs_plan_attention_queries(cfg, cu, grid) == queries
    out, _ = enc.cs_encode(dev_bf16(np.concatenate([c.patches for c in clips])), cu, grid)
    torch.cuda.synchronize()
    row, rows = 0, {}
    for c in clips:
        n = int(c.out_rows.sum())
        # (clips of one length hold the same frames: equal bits wherever they stand in the batch)
        assert torch.equal(rows.setdefault(n, out[row:row + n]), out[row:row + n])
        row += n
        check_items(c.name, c, shared_weights("audio", c), [0])
    assert row == len(out)


def test_small_tiles_of_the_class_token_tower():
    cfg = replace(wl.vit_cls_config(2), tile_patches=(18, 18))
    w = wl.images_workload("tiles_18", cfg, [(252, 252)] * 2, seq_len=2048, data_seed=18)
    assert B.cs_plan_attention_queries(cfg, w.cu_seqlens, w.grid_thw) == 64
    check_items("two tiles of 325 keys", w, w.weights, [0, 1])
