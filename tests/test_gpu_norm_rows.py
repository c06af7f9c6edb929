"""Normalisation kernels on rows of every shape they distinguish: one to eight 16-byte pieces per lane of a wave, the last
piece partly filled; a workgroup per row with pending split-K sums (small batches), and both sides of the row count from
which a wave takes a row alone."""
from dataclasses import replace

import pytest

from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items

pytestmark = pytest.mark.gpu


def vit(hidden):
    return wl.EncoderConfig(arch="vit", dtype="bf16", patch_dim=588, temporal_patch=1, hidden=hidden, n_heads=hidden // 64, head_dim=64,
                            n_layers=2, mlp_dim=512, merger_hidden=256, out_hidden=256, window=8, full_attn_layers=(1,),
                            rope_sections=(0, 16, 16))


# 768: rows of 1536 bytes, the normalised ones and the weights that read them 1664 apart; 192, 256: one piece per lane (48 and 64 of its lanes at work); 320: two of four waves, 1024: all four; 1088: a fifth for
# 16 lanes; 1344: six of eight, 2048: all
@pytest.mark.parametrize("hidden", [192, 256, 320, 768, 1024, 1088, 1344, 2048])
def test_rms_rows(hidden):
    w = wl.images_workload(f"rows_{hidden}", vit(hidden), [(140, 84), (28, 56)], seq_len=512, data_seed=hidden)
    check_items(f"vision tower, hidden {hidden}", w, w.weights, [0, 1])


@pytest.mark.parametrize("hidden", [192, 320, 1088, 1344])
def test_layer_norm_rows(hidden):
    cfg = replace(wl.audio_config(2), hidden=hidden, n_heads=hidden // 64, head_dim=64, mlp_dim=512, out_hidden=256)
    w = wl.audio_workload(f"clip_{hidden}", cfg, 2, 136, seq_len=512, data_seed=hidden)
    check_items(f"audio tower, hidden {hidden}", w, w.weights, [0, 1])


# a LayerNorm tower whose rows are set apart: one tile (split sums, the normalisation kernel writes the rows) and three
# (3084 tokens: the residual GEMMs write them, scaled by the gain, and QKV and fc1 normalise)
@pytest.mark.parametrize("n_tiles", [1, 3])
def test_layer_norm_rows_apart(n_tiles):
    cfg = replace(wl.vit_cls_config(2), hidden=768, n_heads=12, mlp_dim=1536, merger_hidden=512, out_hidden=512)
    w = wl.images_workload(f"tiles_768_{n_tiles}", cfg, [(448, 448)] * n_tiles, seq_len=2048, data_seed=n_tiles)
    check_items(f"class-token tower, hidden 768, {n_tiles} tiles", w, w.weights, sorted({0, n_tiles - 1}))


@pytest.mark.parametrize("size", [(896, 448), (532, 756)])       # 2048 rows, 2052 rows
def test_row_counts(size):
    w = wl.images_workload(f"image_{size}", vit(320), [size], seq_len=1024, data_seed=size[0])
    check_items(f"vision tower, {int(w.cu_seqlens[-1])} rows", w, w.weights, [0])
