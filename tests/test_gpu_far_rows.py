"""cs_linear_bf16 on rows too far apart for 32-bit offsets from a tile's first row: wide and negative pitches, long K."""
import pytest
import torch

from paper_2603_12118_amd import binding as B

DEV = "cuda:0"


@pytest.mark.parametrize("M,N,K,lda,far", [(3, 12, 64, 1 << 31, True), (2, 12, 64, 1 << 30, False), (2, 12, 64, 1 << 31, True),
                                           (300, 64, 64, 8_421_000, False), (300, 64, 64, 12_000_000, True),
                                           (200, 64, 64, -64, True), (1, 64, 64, -64, False),
                                           (1, 8, 300_000_000, 0, False), (1, 8, 310_000_000, 0, True),
                                           (1, 4, 2 ** 31 - 64, 0, True)])
def test_route(M, N, K, lda, far):
    for dtype in ("f32", "bf16"):
        assert ("far rows" in B.cs_linear_kernel(M, N, K, lda, dtype)) == far


def _check(A_ptr, lda, a, w, out):
    """a, w: the values behind the pointers, small whole numbers: products and sums are exact"""
    M, N = out.shape
    B._check(B.lib().cs_linear_bf16(A_ptr, lda, w.data_ptr(), None, out.data_ptr(),
                                    B.CS_BF16 if out.dtype == torch.bfloat16 else B.CS_F32, M, N, w.shape[1], B._stream()))
    torch.cuda.synchronize()
    cols = (w != 0).any(0).nonzero()[:, 0]
    ref = a[:, cols].double().cpu() @ w[:, cols].double().cpu().T
    assert ref.abs().max() <= 256          # whole numbers of eight bits: bf16 holds them too
    assert torch.equal(out.double().cpu(), ref)


def _whole(shape, gen):
    return torch.randint(-2, 3, shape, generator=gen, device=DEV).bfloat16()


# three rows of 4 GiB each with a bf16 output whose rows start 8-byte aligned; the same two-rowed; tiles with ragged edges
@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,lda,dtype", [(3, 12, 64, 1 << 31, torch.bfloat16), (2, 20, 64, 1 << 31, torch.float32),
                                             (300, 140, 64, 12_000_000, torch.float32),
                                             (300, 132, 64, 12_000_000, torch.bfloat16)])
def test_wide_pitch(M, N, K, lda, dtype):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + N)
    store = torch.empty((M - 1) * lda + K, dtype=torch.bfloat16, device=DEV)
    A = store.as_strided((M, K), (lda, 1))
    A.copy_(_whole((M, K), gen))
    out = torch.full((M, N), 7.0, dtype=dtype, device=DEV)
    _check(A.data_ptr(), lda, A, _whole((N, K), gen), out)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(5, 12, 64), (200, 64, 192), (129, 132, 320)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_in_reverse(M, N, K, dtype):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + N + K)
    A = _whole((M, K), gen)
    out = torch.full((M, N), 7.0, dtype=dtype, device=DEV)
    _check(A[M - 1].data_ptr(), -K, A.flip(0), _whole((N, K), gen), out)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [64, 256])      # the rows of W within 4 GiB, and beyond
def test_long_k(N):
    K = 8_421_568
    assert ("far rows" in B.cs_linear_kernel(3, N, K)) == (N == 256)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(N)
    cols = torch.tensor(sorted({0, 63, 64, 1000, K // 2, K - 65, K - 64, K - 1}), device=DEV)
    a, w = torch.zeros(3, K, dtype=torch.bfloat16, device=DEV), torch.zeros(N, K, dtype=torch.bfloat16, device=DEV)
    a[:, cols], w[:, cols] = _whole((3, len(cols)), gen), _whole((N, len(cols)), gen)
    _check(a.data_ptr(), K, a, w, torch.full((3, N), 7.0, device=DEV))
