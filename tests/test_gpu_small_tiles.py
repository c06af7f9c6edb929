"""GEMM launches of at most one round of the chip (64 x 64 up to 128 x 256 tiles, three or four K slices in flight):
edges of every tile, K loops shorter than the pipeline, and the towers' small batches that run on them.  The tiles whose
waves have unequal shares of the W rows (160 columns) are among them."""
import os
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, shared_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,N,tile", [(1, 4, "64, 64"), (63, 60, "64, 64"), (65, 68, "64, 64"), (250, 3836, "64, 64"),
                                      (257, 6000, "64, 128"), (450, 3844, "64, 128"),
                                      (257, 6900, "128, 128"), (520, 3844, "128, 128"), (1000, 3840, "128, 128"),
                                      (1028, 1028 * 3, "128, 128"), (3000, 1280, "128, 128"),
                                      (1030, 4100, "128, 256"), (1500, 3840, "128, 256"), (1500, 5120, "128, 256"),
                                      (8190, 1280, "256, 160")])   # two stages; waves without a share of the last W rows
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 1280])
def test_linear_one_round_tiles(M, N, tile, K):
    assert B.cs_linear_kernel(M, N, K).startswith(f"gemm_kernel<{tile}, ")
    g = torch.Generator(device=DEV)
    g.manual_seed(M * 7 + N * 3 + K)
    A = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    W = torch.randn(N, K, generator=g, device=DEV).bfloat16()
    bias = torch.randn(N, generator=g, device=DEV)
    C = torch.full((M + 1, N), 7.0, device=DEV)
    B.cs_linear_bf16(A, W, bias, C[:M])
    ref = A.float().cpu().double() @ W.float().cpu().double().T + bias.cpu().double()
    err = (C[:M].cpu().double() - ref).abs().max().item()
    # bf16 products are exact in fp32; the sums of K unit-variance products and the bias round at 2^-24 relative to
    # the partial sums, which stay below 8 sqrt(K): K steps at most
    assert err <= K * 2.0 ** -24 * 8 * (K ** 0.5 + 1), err
    assert (C[M] == 7.0).all()


# a residual GEMM on eight-wave 128 x 160 tiles, four stages, of which half the waves load one piece less per slice: the
# out projection's K loop of five slices, and a down projection of one to five
@pytest.mark.parametrize("mlp_dim", [64, 128, 192, 256, 320])
def test_short_k_on_unequal_waves(mlp_dim):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,), hidden=320, n_heads=4, mlp_dim=mlp_dim,
                  merger_hidden=1280, out_hidden=512)
    w = wl.images_workload(f"narrow_{mlp_dim}", cfg, [(308, 364), (56, 84)], seq_len=2048, data_seed=mlp_dim)
    enc = B.Encoder(cfg, w.weights)
    for step in ("proj", "mlp_down") if not any(k.startswith("CS_GEMM_") for k in os.environ) else ():
        assert enc.cs_encoder_step_kernel(B.STEPS[step], int(w.cu_seqlens[-1])).startswith("gemm_kernel<128, 160, 4, 2, 4, 0>")
    check_items(f"hidden 320, mlp {mlp_dim}", w, w.weights, [0, 1])


@pytest.mark.parametrize("sizes", [[(28, 28)], [(56, 84)], [(224, 224)], [(308, 364)], [(224, 224), (336, 420)], [(448, 448)]])
def test_small_image_batches(sizes):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"small_{len(sizes)}", cfg, sizes, seq_len=2048, data_seed=sum(h + w_ for h, w_ in sizes))
    W = shared_weights("vit", w)
    check_items(f"images {sizes}", w, W, list(range(len(sizes))))


@pytest.mark.parametrize("n_clips,frames", [(1, 64), (1, 1000), (1, 3000), (2, 1208)])
def test_small_audio_batches(n_clips, frames):
    w = wl.audio_workload(f"small_audio_{n_clips}x{frames}", wl.audio_config(2), n_clips, frames, seq_len=2048, data_seed=frames)
    W = shared_weights("audio", w)
    check_items(f"audio {n_clips} x {frames}", w, W, [n_clips - 1])


def test_one_tile_of_the_class_token_tower():
    w = wl.images_workload("tile", wl.vit_cls_config(2), [(448, 448)], seq_len=2048, data_seed=5)
    W = shared_weights("cls", w)
    check_items("one tile", w, W, [0])
