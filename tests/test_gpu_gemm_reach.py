"""rose_gemm_bf16 with operands that 32-bit offsets do not span, each against
the exact product of the BF16-rounded operands (bound as in
test_gpu_gemm.py): row pitches of 2^21 and 2^24 elements on either side and
along k, negative strides, and operands of more than 2 GiB; with remainders
in m, n and k.  The bits equal those of the same values held contiguously."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _gemm(M, N, K, A, sa, B, sb):
    """A, B: pointers to element (0, 0); sa, sb: their strides."""
    from paper_2105_05600_amd import rose
    C = torch.empty((M, N), device="cuda")
    rose._check("rose_gemm_bf16", rose._lib.rose_gemm_bf16(M, N, K, A, sa[0], sa[1], B, sb[0], sb[1], rose._ptr(C), N,
                                                           rose._stream()))
    return C


def _check(M, N, K, a, b, C):
    from paper_2105_05600_amd import rose
    assert torch.equal(C, rose.gemm_bf16(a.contiguous(), b.contiguous()))
    x, y = a.bfloat16().double(), b.bfloat16().double()
    assert bool(((C.double() - x @ y).abs() <= 2.0 * K * 2.0 ** -24 * (x.abs() @ y.abs())).all())


def _spread(rows, cols, pitch, axis, g):
    """A rows x cols matrix whose `axis` has the pitch, the other one is contiguous."""
    n, m = (rows, cols) if axis == 0 else (cols, rows)
    buf = torch.empty((n - 1) * pitch + m, device="cuda")
    v = buf.as_strided((n, m), (pitch, 1))
    v.copy_(torch.randn((n, m), generator=g, device="cuda"))
    return v if axis == 0 else v.t()


@pytest.mark.parametrize("pitch", [1 << 21, 1 << 24])
@pytest.mark.parametrize("which,axis", [("a", 0), ("a", 1), ("b", 0), ("b", 1)])
def test_pitches(which, axis, pitch):
    from paper_2105_05600_amd import rose
    g = torch.Generator(device="cuda").manual_seed(pitch + axis)
    other = 531 if pitch < 1 << 24 else 45  # 64 x 64 tiles, or the small kernel
    # the axis with the pitch has 33 or 35 entries, the others remainders
    M, K = (33, 517) if axis == 0 else (other, 35)
    if which == "a":
        A = _spread(M, K, pitch, axis, g)
        B = torch.randn((K, other * 13), generator=g, device="cuda")
    else:
        N, K = (33, 517) if axis == 1 else (other, 35)
        A = torch.randn((other * 13, K), generator=g, device="cuda")
        B = _spread(K, N, pitch, axis, g)
    _check(A.shape[0], B.shape[1], A.shape[1], A, B, rose.gemm_bf16(A, B))


@pytest.mark.parametrize("M,N,K", [(37, 45, 300), (1030, 777, 70), (2050, 2049, 515)])
@pytest.mark.parametrize("flip", ["a0", "a1", "b0", "b1"])
def test_negative_strides(M, N, K, flip):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, b = torch.randn((M, K), generator=g, device="cuda"), torch.randn((K, N), generator=g, device="cuda")
    pa, sa, pb, sb = a.data_ptr(), [K, 1], b.data_ptr(), [N, 1]
    d = int(flip[1])
    if flip[0] == "a":
        pa, sa[d] = pa + 4 * sa[d] * (a.shape[d] - 1), -sa[d]
        C = _gemm(M, N, K, pa, sa, pb, sb)
        a = a.flip(d)
    else:
        pb, sb[d] = pb + 4 * sb[d] * (b.shape[d] - 1), -sb[d]
        C = _gemm(M, N, K, pa, sa, pb, sb)
        b = b.flip(d)
    _check(M, N, K, a, b, C)


@pytest.mark.parametrize("M,N,K,which", [(5, 65531, 8230, "b"), (261, 32768, 16400, "b"), (65530, 70, 8220, "a")])
def test_operands_past_2_gib(M, N, K, which):
    """Row-major B, or column-major A: k steps by the long dimension."""
    from paper_2105_05600_amd import rose
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((M, K) if which == "b" else (K, M), generator=g, device="cuda")
    B = torch.randn((K, N), generator=g, device="cuda")
    if which == "a":
        A = A.t()
    assert 4 * max(A.numel(), B.numel()) > 2 ** 31
    C = rose.gemm_bf16(A, B)
    # rows and columns at the ends, in binary64
    rows = torch.tensor(sorted({0, M // 2, M - 1}), device="cuda")
    cols = torch.tensor(sorted({0, 1, N // 2, N - 33, N - 1}), device="cuda")
    x, y = A[rows].bfloat16().double(), B[:, cols].bfloat16().double()
    err = (C[rows][:, cols].double() - x @ y).abs()
    assert bool((err <= 2.0 * K * 2.0 ** -24 * (x.abs() @ y.abs())).all())


def test_a_product_past_2_gib_takes_the_time_of_its_halves():
    """It runs on the same kernels: at most twice the time of the two halves in k, which lie below 2 GiB."""
    from paper_2105_05600_amd import rose
    M, N, K = 256, 32768, 17408
    A, B = torch.randn((M, K), device="cuda"), torch.randn((K, N), device="cuda")

    def best(*parts):
        t = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for a, b in parts:
                rose.gemm_bf16(a, b)
            e1.record()
            e1.synchronize()
            t.append(e0.elapsed_time(e1))
        return min(t)

    h = K // 2
    assert best((A, B)) < 2.0 * best((A[:, :h], B[:h]), (A[:, h:], B[h:]))
