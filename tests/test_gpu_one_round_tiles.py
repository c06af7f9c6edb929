"""Launches that the chip holds in one round: 192 x 256 tiles, where 128 x 256 need more than one, residual GEMMs on 64 x 160
and 192 x 160 tiles, and the class-token tower's in parts over K.  Both ends of each range, ragged last tiles of either
direction, and K loops as short as one slice."""
import os
from dataclasses import replace

import pytest
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, shared_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def runs(cfg, W, n_tokens, **kernels):
    if any(k.startswith("CS_") for k in os.environ):
        return
    enc = B.Encoder(cfg, W)
    for step, kernel in kernels.items():
        assert enc.cs_encoder_batch_kernel(B.STEPS[step], n_tokens) == kernel, (step, n_tokens)


# 27 column tiles, the last of 256 or 244 columns: 1153 rows (seven tile rows, the last of one row) to 1728 (nine full ones), and
# one more; 15 column tiles, the last of 4 columns: 3264 rows are seventeen full tile rows and 255 tiles; and fewer
@pytest.mark.parametrize("M,N,tile", [(1153, 6912, "192, 256"), (1728, 6900, "192, 256"), (1729, 6900, "256, 256"), (2177, 3588, "192, 256"),
                                      (3264, 3588, "192, 256"), (2561, 3840, "192, 256"), (2560, 3840, "256, 160")])
@pytest.mark.parametrize("K", [64, 128, 192, 1280])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_linear(M, N, tile, K, dtype):
    if not any(k.startswith("CS_") for k in os.environ):
        assert B.cs_linear_kernel(M, N, K, 0, "bf16" if dtype == torch.bfloat16 else "f32").startswith(f"gemm_kernel<{tile}, ")
    g = torch.Generator(device=DEV)
    g.manual_seed(M * 7 + N * 3 + K)
    A = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    W = torch.randn(N, K, generator=g, device=DEV).bfloat16()
    bias = torch.randn(N, generator=g, device=DEV)
    C = torch.full((M + 1, N), 7.0, device=DEV, dtype=dtype)
    B.cs_linear_bf16(A, W, bias, C[:M])
    ref = A.double() @ W.double().T + bias.double()
    # bf16 products are exact in fp32; the sums of K unit-variance products and the bias round at 2^-24 relative to the
    # partial sums, which stay below 8 sqrt(K): K steps at most; a bf16 result rounds once more, 2^-9 of itself
    bound = K * 2.0 ** -24 * 8 * (K ** 0.5 + 1) + (ref.abs() * 2.0 ** -8 if dtype == torch.bfloat16 else 0)
    assert ((C[:M].double() - ref).abs() <= bound).all()
    assert (C[M] == 7.0).all()


SWIGLU_192, QKV_192, GELU_192 = (f"gemm_kernel<192, 256, 2, 4, {epi}, 0> 16x16x32" for epi in (5, 6, 2))   # (QKV: of a tower without a rotary embedding)
PROJ_64 = "gemm_kernel<64, 160, 2, 2, 4, 0> 16x16x32"


# gate|up: 1156 tokens (a last tile row of four) and 1728; the out projection: 1924 tokens, not
# split any more, and 2048, the most that 64 x 160 tiles take; QKV: 2392 tokens are thirteen tile rows of 192 x 256
@pytest.mark.parametrize("sizes,kernels", [([(476, 476)], dict(mlp_up=SWIGLU_192)), ([(504, 672)], dict(mlp_up=SWIGLU_192)),
                                           ([(448, 840), (28, 28)], dict(proj=PROJ_64)),
                                           ([(448, 896)], dict(proj=PROJ_64)), ([(644, 728)], dict(qkv=QKV_192 + ", 128 positions"))])
def test_images(sizes, kernels):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"one_round_{len(sizes)}_{sizes[0][1]}", cfg, sizes, seq_len=2048, data_seed=sizes[0][1])
    W = shared_weights("vit", w)
    runs(cfg, W, int(w.cu_seqlens[-1]), **kernels)
    check_items(f"{int(w.cu_seqlens[-1])} tokens", w, W, sorted({0, len(sizes) - 1}))


# down projections of one to four slices (the pipeline holds four) at both ends of the rows that take 64 x 160 tiles
@pytest.mark.parametrize("mlp_dim", [64, 128, 192, 256])
@pytest.mark.parametrize("sizes", [[(420, 420), (112, 112)], [(448, 868), (84, 140)]])
def test_short_k_on_64_rows(sizes, mlp_dim):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(), hidden=1280, n_heads=16, mlp_dim=mlp_dim, merger_hidden=512, out_hidden=512)
    w = wl.images_workload(f"short_64_{sizes[0][1]}_{mlp_dim}", cfg, sizes, seq_len=2048, data_seed=mlp_dim)
    runs(cfg, w.weights, int(w.cu_seqlens[-1]), mlp_down=PROJ_64)
    check_items(f"{int(w.cu_seqlens[-1])} tokens, mlp {mlp_dim}", w, w.weights, [0, 1])


# a narrow tower's, which also write the plain sums of the folded LayerNorm: two column tiles of 65 tile rows, and one and
# five slices
@pytest.mark.parametrize("mlp_dim", [64, 320])
def test_narrow_clips_on_64_rows(mlp_dim):
    cfg = replace(wl.audio_config(2), attn_chunk=100, hidden=320, n_heads=5, mlp_dim=mlp_dim, out_hidden=512)
    w = wl.audio_workload(f"narrow_64_{mlp_dim}", cfg, 5, 1640, seq_len=2048, data_seed=mlp_dim)
    runs(cfg, w.weights, 4100, proj=PROJ_64.replace("4, 0>", "9, 0>"), mlp_down=PROJ_64.replace("4, 0>", "9, 0>"))
    check_items(f"five clips of 820 tokens, mlp {mlp_dim}", w, w.weights, [0, 4])


# The launches in front of the blocks and behind them, on 192 x 256 tiles as the plain ones of their sizes: the first
# convolution (GELU, a row map) and the second (fp32 GELU, rows between the clips that belong to neither), the patch embeddings, and
# the merger's first product (GELU into a high and a low half)
def plain_192(*shapes):
    if not any(k.startswith("CS_") for k in os.environ):
        for shape in shapes:
            assert B.cs_linear_kernel(*shape) == "gemm_kernel<192, 256, 2, 4, 1, 0> 16x16x32", shape


@pytest.mark.parametrize("n_clips,frames", [(3, 2800), (7, 2400)])   # 8400 frames; 8400 tokens
def test_convolutions_on_192_rows(n_clips, frames):
    plain_192((8400, 1280, 384), (8406, 1280, 3840))
    w = wl.audio_workload(f"convolutions_192_{n_clips}", replace(wl.audio_config(1), attn_chunk=100), n_clips, frames, seq_len=2048, data_seed=n_clips)
    check_items(f"{n_clips} clips of {frames} frames", w, shared_weights("audio_1", w), [0, n_clips - 1])


# (at 2305 merge groups it is the merger's second product, whose rows go to their places through a map)
@pytest.mark.parametrize("n,merger", [(8, (2049, 5120, 2 * 5120)), (9, (2305, 3584, 2 * 5120))])
def test_patches_and_merger_on_192_rows(n, merger):
    plain_192((1024 * n + 4, 1280, 1216), merger)
    cfg = replace(wl.vit_7b_config(1), dtype="bf16", full_attn_layers=())
    w = wl.images_workload(f"merger_192_{n}", cfg, [(448, 448)] * n + [(28, 28)], seq_len=2048, data_seed=n)
    check_items(f"{1024 * n + 4} patches", w, shared_weights("vit_1", w), [0, n])


def test_nine_class_token_tiles():
    plain_192((9 * 1028, 1024, 640), (9 * 257, 4096, 2 * 4096))
    w = wl.images_workload("nine_tiles", wl.vit_cls_config(1), [(448, 448)] * 9, seq_len=2048, data_seed=9)
    check_items("nine tiles", w, shared_weights("cls_1", w), [0, 8])


# residual GEMMs on 192 x 160 tiles, six waves: 4100 tokens (the last tile row of 68), 5760, 30 full tile rows,
# and clips of 5140
RES_192 = "gemm_kernel<192, 160, 3, 2, 4, 0> 16x16x32"


@pytest.mark.parametrize("sizes", [[(448, 448)] * 4 + [(28, 28)], [(448, 448)] * 5 + [(448, 280)]])
def test_images_on_192_rows(sizes):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"rows_192_{len(sizes)}_{sizes[-1][0]}", cfg, sizes, seq_len=2048, data_seed=len(sizes))
    W = shared_weights("vit", w)
    runs(cfg, W, int(w.cu_seqlens[-1]), proj=RES_192, mlp_down=RES_192)
    check_items(f"{int(w.cu_seqlens[-1])} tokens", w, W, [0, len(sizes) - 1])


def test_clips_on_192_rows():
    w = wl.audio_workload("rows_192", replace(wl.audio_config(2), attn_chunk=100), 5, 2048 + 8, seq_len=2048, data_seed=6)
    W = shared_weights("audio", w)
    runs(w.cfg, W, 5140, proj=RES_192.replace("4, 0>", "9, 0>"), mlp_down=RES_192.replace("4, 0>", "9, 0>"))
    check_items("five clips of 1028 tokens", w, W, [0, 4])


# down projections of one to ten slices: K loops about as long as the pipeline of three
@pytest.mark.parametrize("mlp_dim", [64, 128, 192, 640])
def test_short_k_on_192_rows(mlp_dim):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(), hidden=1280, n_heads=16, mlp_dim=mlp_dim, merger_hidden=512, out_hidden=512)
    w = wl.images_workload(f"short_192_{mlp_dim}", cfg, [(448, 448)] * 4 + [(28, 56)], seq_len=2048, data_seed=mlp_dim)
    runs(cfg, w.weights, int(w.cu_seqlens[-1]), mlp_down=RES_192)
    check_items(f"mlp {mlp_dim}", w, w.weights, [0, 4])


# fc1 and QKV of two clips (2200 tokens)
def test_two_clips():
    cfg = replace(wl.audio_config(2), attn_chunk=200)
    w = wl.audio_workload("one_round_2x2200", cfg, 2, 2200, seq_len=2048, data_seed=2)
    W = shared_weights("audio", w)
    runs(cfg, W, 2200, mlp_up=GELU_192, qkv=QKV_192)
    check_items("two clips of 1100 tokens", w, W, [1])


# 16 slices in two parts and 64 in three (21, 21 and 22) or two
@pytest.mark.parametrize("tiles,proj,down", [(1, 2, 3), (2, 2, 2)])
def test_class_token_tiles(tiles, proj, down):
    w = wl.images_workload(f"one_round_tiles_{tiles}", wl.vit_cls_config(2), [(448, 448)] * tiles, seq_len=2048, data_seed=tiles)
    W = shared_weights("cls", w)
    if not any(k.startswith("CS_") for k in os.environ):
        enc = B.Encoder(w.cfg, W)
        for step, parts in (("proj", proj), ("mlp_down", down)):
            assert enc.cs_encoder_batch_kernel(B.STEPS[step], 1028 * tiles).endswith(f", K in {parts} parts")
    check_items(f"{tiles} tiles", w, W, [tiles - 1])
