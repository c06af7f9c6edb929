"""One-round launches on 128 x 160 tiles (plain, GELU and split-K epilogues): column counts that fill the last tile to any
number of 32-column blocks, ragged rows, K loops shorter than the pipeline, and the shapes just beyond the rule."""
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


# the towers' launches of that kind: GELU of a LayerNorm tower (one tile; clips of 600 to 1000 tokens), the merger and
# four-part residual GEMMs
def test_one_tile():
    w = wl.images_workload("tile", wl.vit_cls_config(2), [(448, 448)], seq_len=2048, data_seed=5)
    check_items("one tile", w, shared_weights("cls", w), [0])


@pytest.mark.parametrize("frames", [1208, 2000])
def test_one_clip(frames):
    w = wl.audio_workload(f"clip_{frames}", replace(wl.audio_config(2), attn_chunk=100), 1, frames, seq_len=2048, data_seed=frames)
    check_items(f"clip of {frames // 2} tokens", w, shared_weights("audio", w), [0])


def test_one_image():
    cfg = replace(wl.vit_7b_config(2), dtype="bf16", full_attn_layers=(1,))
    w = wl.images_workload("image", cfg, [(420, 448)], seq_len=2048, data_seed=3)
    check_items("one image of 960 patches", w, shared_weights("vit", w), [0])
