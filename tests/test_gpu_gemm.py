"""rose_gemm_bf16 at the edges of its kernels (32 x 32 tiles; 64 x 64, 128 x
128 and 256 x 256 tiles for larger outputs) and of their k-steps, for operands
stored along k, along their rows, with a row pitch and with general strides:
against the exact products of the BF16-rounded operands in binary64.  The
binary32 accumulation of K products is off by at most K 2^-24 sum |a b| (each
partial sum rounded once), doubled here for the instruction's inner sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _operand(rows, cols, how, g):
    """A rows x cols matrix held as asked: 'rm' row-major, 'cm' column-major,
    'pitch' row-major with a longer row, 'odd' every second column of a
    wider matrix that starts 4 bytes off a 16-byte line."""
    if how == "rm":
        return torch.randn((rows, cols), generator=g, device="cuda")
    if how == "cm":
        return torch.randn((cols, rows), generator=g, device="cuda").t()
    if how == "pitch":
        return torch.randn((rows, cols + 3), generator=g, device="cuda")[:, 1:cols + 1]
    return torch.randn((rows, 2 * cols + 1), generator=g, device="cuda")[:, 1::2]


SHAPES = [(1, 1, 1), (1, 12, 7), (33, 31, 17), (32, 32, 256), (31, 65, 257), (1024, 12, 512), (1216, 256, 1024),
          # 64 x 64 tiles: 192 of them or more, with remainders in m, n and k
          (1024, 768, 64), (961, 769, 33), (2047, 400, 300),
          # 128 x 128 tiles: 256 or more and K of 512 or more
          (2048, 2048, 512), (1921, 2049, 513), (3841, 1025, 530),
          # 256 x 256 tiles: 192 or more
          (4096, 3072, 512), (3841, 3073, 527), (3585, 3329, 540)]


@pytest.mark.parametrize("a_how,b_how", [("rm", "rm"), ("cm", "rm"), ("rm", "cm"), ("cm", "cm"), ("pitch", "pitch"),
                                         ("odd", "odd")])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_edges(M, N, K, a_how, b_how):
    from paper_2105_05600_amd import rose
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N * 3 + K)
    A, B = _operand(M, K, a_how, g), _operand(K, N, b_how, g)
    C = rose.gemm_bf16(A, B)
    a, b = A.bfloat16().double(), B.bfloat16().double()
    ref, mag = a @ b, a.abs() @ b.abs()
    bound = 2.0 * K * 2.0 ** -24 * mag
    assert bool(((C.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("M,N,K", [(64, 64, 300), (1024, 1024, 300), (2048, 2048, 600), (4096, 3072, 600)])
def test_gemm_infinities_and_nan(M, N, K):
    from paper_2105_05600_amd import rose
    g = torch.Generator(device="cuda").manual_seed(5)
    A, B = _operand(M, K, "rm", g).abs() + 0.5, _operand(K, N, "rm", g).abs() + 0.5
    A[3, 5], A[M - 1, K - 1], A[7, 2] = float("inf"), float("nan"), -float("inf")
    A[9, 1] = 3.4028234e38  # rounds up to infinity in bfloat16
    C = rose.gemm_bf16(A, B)
    assert bool((C[3] == float("inf")).all()) and bool(C[M - 1].isnan().all())
    assert bool((C[7] == -float("inf")).all()) and bool((C[9] == float("inf")).all())
    rest = torch.ones(M, dtype=torch.bool, device="cuda")
    rest[[3, 7, 9, M - 1]] = False
    assert bool(C[rest].isfinite().all())
