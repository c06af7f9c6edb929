"""GEMM launches of at most one round of the chip (64 x 64 up to 128 x 256 tiles, three or four K slices in flight):
edges of every tile, K loops shorter than the pipeline, and the towers' small batches that run on them."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, shared_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,N", [(1, 4), (63, 60), (65, 68), (250, 3836),        # 64 x 64 tiles
                                 (257, 6900), (520, 3844),                       # 64 x 128
                                 (1000, 3840), (1028, 1028 * 3),                 # 128 x 128
                                 (1030, 4100), (1500, 3840),                     # 128 x 256
                                 (1500, 5120), (3000, 1280)])                    # 256 x 160: a wave without a share of the last W rows
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 1280])
def test_linear_one_round_tiles(M, N, K):
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
