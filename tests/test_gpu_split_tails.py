"""256 x 256 launches whose last round is cut into half tiles beside 64-row tiles for the rows of a ragged last tile row:
one tile to cut and half a round of them, remainders from one group of rows to almost a tile, and the counts at which the
halves and the light tiles no longer make one round."""
import os
from dataclasses import replace

import pytest
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, shared_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# full tiles of N / 256 columns each: 17 x 16 = 272 (16 to cut), 52 x 5 = 260, 24 x 16 = 384 (128 to cut: 256 halves leave no
# room for light tiles, so none are cut), 23 x 16 = 368 (112 to cut; 224 halves and 16 or 64 light tiles), 20 x 15 = 300
@pytest.mark.parametrize("full_rows,N,halves", [(17, 4096, 32), (24, 4096, 0), (23, 4096, 224), (20, 3840, 88), (52, 1276, 8)])
@pytest.mark.parametrize("rest", [1, 64, 65, 255])
@pytest.mark.parametrize("K", [64, 192])
def test_halves_beside_light_tiles(full_rows, N, halves, rest, K):
    M = full_rows * 256 + rest
    if halves + (rest + 63) // 64 * -(-N // 256) > 256:   # halves and light tiles would not make one round
        halves = 0
    if not any(k.startswith("CS_GEMM_") for k in os.environ):
        assert B.cs_linear_kernel(M, N, K) == "gemm_kernel<256, 256, 2, 4, 1, 1> 16x16x32" + (f", {halves} half tiles" if halves else "")
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    A = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    W = torch.randn(N, K, generator=g, device=DEV).bfloat16()
    bias = torch.randn(N, generator=g, device=DEV)
    C = torch.full((M + 1, N), 7.0, device=DEV)
    B.cs_linear_bf16(A, W, bias, C[:M])
    ref = A.double() @ W.double().T + bias.double()
    err = (C[:M].double() - ref).abs().max().item()
    # bf16 products are exact in fp32; the sums of K unit-variance products and the bias round at 2^-24 relative to the
    # partial sums, which stay below 8 sqrt(K): K steps at most
    assert err <= K * 2.0 ** -24 * 8 * (K ** 0.5 + 1), err
    assert (C[M] == 7.0).all()


# the vision tower's launches of that kind: QKV with rotary behind a folded RMSNorm (4936 tokens: 19 x 15 whole tiles, 72 rows
# behind them) and the merger's hi | lo GELU (14 140 tokens, 3535 groups: 13 x 20 whole tiles, 207 rows)
@pytest.mark.parametrize("sizes", [[(448, 448)] * 4 + [(364, 448), (28, 56)], [(448, 448)] * 13 + [(252, 644)]])
def test_images(sizes):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"images_{len(sizes)}", cfg, sizes, seq_len=16384, data_seed=len(sizes))
    W = shared_weights("vit", w)
    if len(sizes) == 6 and not any(k.startswith("CS_GEMM_") for k in os.environ):
        assert B.Encoder(cfg, W).cs_encoder_step_kernel(B.STEPS["qkv"], 4936) == "gemm_kernel<256, 256, 2, 4, 6, 1> 16x16x32, 58 half tiles"
    check_items(f"{int(w.cu_seqlens[-1])} patches", w, W, [0, len(sizes) - 1])
