"""256 x 256 launches whose last round is cut into half tiles beside 64-row tiles for the rows of a ragged last tile row:
one tile to cut and half a round of them, remainders from one group of rows to almost a tile, and the counts at which the
halves and the light tiles no longer make one round."""
import pytest
import torch

from paper_2603_12118_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# full tiles of N / 256 columns each: 17 x 16 = 272 (16 to cut), 52 x 5 = 260, 24 x 16 = 384 (128 to cut: 256 halves leave no
# room for light tiles, so none are cut), 23 x 16 = 368 (112 to cut; 224 halves and 16 or 64 light tiles), 20 x 15 = 300
@pytest.mark.parametrize("full_rows,N", [(17, 4096), (24, 4096), (23, 4096), (20, 3840), (52, 1276)])
@pytest.mark.parametrize("rest", [1, 64, 65, 255])
@pytest.mark.parametrize("K", [64, 192])
def test_halves_beside_light_tiles(full_rows, N, rest, K):
    M = full_rows * 256 + rest
    assert B.cs_linear_kernel(M, N, K).startswith("gemm_kernel<256, 256, 2, 4, ")
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
