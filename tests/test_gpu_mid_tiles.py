"""One-round launches on 128 x 160 tiles (plain, GELU, hi | lo GELU and split-K epilogues): column counts that fill the last tile to any
number of 32-column blocks, ragged rows, K loops shorter than the pipeline, and the shapes just beyond the rule."""
import os
from dataclasses import replace

import pytest
import torch

from paper_2603_12118_amd import binding as B
from paper_2603_12118_amd import workloads as wl
from tests.test_gpu_batch_sizes import check_items, shared_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 24 column tiles and one of 32, 64, 96 or 128 columns; 256 workgroups exactly, and one tile row more; a column count that
# is no multiple of 32
@pytest.mark.parametrize("M,N,tile", [(1030, 3840, "128, 160"), (1152, 3872, "128, 160"), (1025, 3904, "128, 160"), (1100, 3936, "128, 160"),
                                      (1028, 3968, "128, 160"), (1024, 5120, "128, 160"), (1025, 5120, "128, 256"), (1030, 3844, "128, 256")])
@pytest.mark.parametrize("K", [64, 192, 256, 1280])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_linear(M, N, tile, K, dtype):
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


# The towers' launches of that kind.  One tile, clips of 804 and 1000 tokens: fc1 with GELU, four-part residual GEMMs
def test_one_tile():
    w = wl.images_workload("tile", wl.vit_cls_config(2), [(448, 448)], seq_len=2048, data_seed=5)
    check_items("one tile", w, shared_weights("cls", w), [0])


@pytest.mark.parametrize("frames", [1608, 2000])
def test_one_clip(frames):
    w = wl.audio_workload(f"clip_{frames}", replace(wl.audio_config(2), attn_chunk=100), 1, frames, seq_len=2048, data_seed=frames)
    W = shared_weights("audio", w)
    if not any(k.startswith("CS_GEMM_") for k in os.environ):
        assert B.Encoder(w.cfg, W).cs_encoder_step_kernel(B.STEPS["mlp_up"], frames // 2).startswith("gemm_kernel<128, 160, 4, 2, 2, 0>")
    check_items(f"clip of {frames // 2} tokens", w, W, [0])


# first convolution of one clip (3400 rows, GELU and a row map), second convolution of two (3401 rows, of which one belongs
# to neither, fp32 GELU); fc1 of the latter runs half tiles beside 64-row tiles behind a folded LayerNorm (13 x 20 whole
# tiles and 72 rows)
@pytest.mark.parametrize("n_clips", [1, 2])
def test_convolutions(n_clips):
    w = wl.audio_workload(f"clips_{n_clips}", replace(wl.audio_config(2), attn_chunk=200), n_clips, 3400, seq_len=4096, data_seed=n_clips)
    W = shared_weights("audio", w)
    if n_clips == 2 and not any(k.startswith("CS_GEMM_") for k in os.environ):
        name = B.Encoder(w.cfg, W).cs_encoder_step_kernel(B.STEPS["mlp_up"], 3400)
        assert name == "gemm_kernel<256, 256, 2, 4, 2, 1> 16x16x32, 8 half tiles"
    check_items(f"{n_clips} clips of 1700 tokens", w, W, sorted({0, n_clips - 1}))


# patch embedding and merger of batches too large for split sums: 975 and 775 merge groups (last tile rows of 79 and 7);
# four tiles of the class-token tower, 1028 groups and a last column tile of 96
@pytest.mark.parametrize("last", [(252, 644), (14 * 2, 14 * 14)])
def test_merger_of_images(last):
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload(f"merger_{last}", cfg, [(448, 448)] * 3 + [last], seq_len=2048, data_seed=last[1])
    check_items(f"{int(w.cu_seqlens[-1])} patches", w, shared_weights("vit", w), [0, 3])


def test_merger_of_four_tiles():
    w = wl.images_workload("four_tiles", wl.vit_cls_config(2), [(448, 448)] * 4, seq_len=2048, data_seed=4)
    check_items("four tiles", w, shared_weights("cls", w), [0, 3])


def test_one_image():
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload("image", cfg, [(420, 448)], seq_len=2048, data_seed=3)
    check_items("one image of 960 patches", w, shared_weights("vit", w), [0])
