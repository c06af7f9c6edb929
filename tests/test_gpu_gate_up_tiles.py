"""gate|up of small batches on 128 x 256 tiles: both ends of their range of rows, ragged last tiles of either direction, and
K loops shorter than the pipeline of three slices."""
import os
from dataclasses import replace

import pytest

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, shared_weights

pytestmark = pytest.mark.gpu


def runs(cfg, W, n_tokens, kernel):
    if not any(k.startswith("CS_GEMM_") for k in os.environ):
        assert B.Encoder(cfg, W).cs_encoder_batch_kernel(B.STEPS["mlp_up"], n_tokens) == f"gemm_kernel<{kernel}> 16x16x32"


# 27 column tiles of 256: 512 tokens are one round of 128 x 128 tiles, 516 are not, 1152 are nine tile rows of 128 x 256, and
# 1156 a tenth, which makes more than a round: seven of 192 x 256
@pytest.mark.parametrize("sizes,kernel", [([(448, 224)], "128, 128, 4, 2, 5, 0"), ([(448, 224), (28, 28)], "128, 256, 2, 4, 5, 0"),
                                          ([(448, 504)], "128, 256, 2, 4, 5, 0"), ([(476, 476)], "192, 256, 2, 4, 5, 0")])
def test_rows(sizes, kernel):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"rows_{len(sizes)}_{sizes[0][1]}", cfg, sizes, seq_len=2048, data_seed=sizes[0][1])
    W = shared_weights("vit", w)
    runs(cfg, W, int(w.cu_seqlens[-1]), kernel)
    check_items(f"{int(w.cu_seqlens[-1])} tokens", w, W, list(range(len(sizes))))


# a last column tile of 128, 64 and 256 of its 256 columns, and one to five K slices
@pytest.mark.parametrize("mlp_dim,heads", [(1984, 1), (1952, 2), (2048, 3), (2000, 4), (1984, 5)])
def test_columns_and_short_k(mlp_dim, heads):
    cfg = replace(wl.vit_7b_config(1), dtype="bf16", full_attn_layers=(), hidden=64 * heads, n_heads=heads, head_dim=64,
                  rope_sections=(0, 16, 16), mlp_dim=mlp_dim, merger_hidden=512, out_hidden=512)
    w = wl.images_workload(f"columns_{mlp_dim}", cfg, [(420, 504), (28, 56)], seq_len=2048, data_seed=mlp_dim)
    runs(cfg, w.weights, int(w.cu_seqlens[-1]), "128, 256, 2, 4, 5, 0")
    check_items(f"mlp {mlp_dim}, hidden {64 * heads}", w, w.weights, [0, 1])
