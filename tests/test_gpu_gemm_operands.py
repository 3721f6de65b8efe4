"""Operands of the matrix product beyond the tight, small ones: rows longer than the matrix, operands of 3 GB, outputs that
are stored past the caches.  Whole numbers: exact in any order."""
import pytest

pytestmark = pytest.mark.gpu


def _gemm(a_kc, b_kc, A, lda, B, ldb, M, N, K, C, ldc, tile, split, scratch):
    import torch
    from paper_2201_05500_amd import binding_mlp as BM
    return BM.ctr_debug_mlp_gemm(a_kc, b_kc, A.data_ptr(), lda, B.data_ptr(), ldb, M, N, K, C.data_ptr(), ldc,
                                 scratch.data_ptr(), scratch.numel() * 4, tile, split, torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("tile,split", [(64, 0), (64, 1), (128, 0), (128, 1), (256, 1)])
@pytest.mark.parametrize("a_kc,b_kc", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,K", [(72, 8, 8), (264, 392, 456), (128, 256, 64), (2312, 2568, 72)])
def test_what_lies_behind_the_rows_is_not_read_into_the_product(M, N, K, a_kc, b_kc, tile, split):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M + K)
    ints = lambda shape: torch.randint(-8, 9, shape, generator=gen, device="cuda:0")
    a, b = ints((M, K)), ints((K, N))

    def padded(t):  # NaN behind every row; rows and nothing else up to the end of the allocation
        p = torch.full((t.shape[0], t.shape[1] + 24), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        p[:, :t.shape[1]] = t.to(torch.bfloat16)
        return p
    A, B = padded(a if a_kc else a.t()), padded(b.t() if b_kc else b)
    C = torch.full((M, N + 8), -1.0, device="cuda:0")
    scratch = torch.empty(8 << 20, device="cuda:0")
    assert _gemm(a_kc, b_kc, A, A.shape[1], B, B.shape[1], M, N, K, C, N + 8, tile, split, scratch) == 0
    assert torch.equal(C[:, :N], torch.matmul(a.double(), b.double()).float())
    assert bool((C[:, N:] == -1.0).all())


@pytest.mark.parametrize("a_kc", [True, False])
@pytest.mark.parametrize("tile", [64, 128, 256])
def test_operand_of_three_gigabytes(a_kc, tile):
    import torch
    M, N, K = (1 << 20, 8, 1544) if a_kc else (1536, 8, (1 << 20) + 8)
    A = torch.zeros((M, K) if a_kc else (K, M), dtype=torch.bfloat16, device="cuda:0")
    assert 3 << 30 < A.numel() * 2 < 4 << 30
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tile)
    last = torch.randint(-8, 9, (264, A.shape[1]), generator=gen, device="cuda:0")
    A[-264:] = last.to(torch.bfloat16)
    b = torch.randint(-8, 9, (K, N), generator=gen, device="cuda:0")
    B = b.to(torch.bfloat16)
    C = torch.full((M, N), -1.0, device="cuda:0")
    scratch = torch.empty(8, device="cuda:0")  # no room: one range
    assert _gemm(a_kc, False, A, A.shape[1], B, N, M, N, K, C, N, tile, 0, scratch) == 0
    if a_kc:
        assert torch.equal(C[-264:], torch.matmul(last.double(), b.double()).float()) and not bool(C[:-264].any())
    else:
        assert torch.equal(C, torch.matmul(last.t().double(), b[-264:].double()).float())


@pytest.mark.parametrize("N", [8192, 8200])
def test_output_larger_than_the_caches(N):
    import torch
    M, K = 8200, 136
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(N)
    a = torch.randint(-8, 9, (M, K), generator=gen, device="cuda:0").float()
    b = torch.randint(-8, 9, (N, K), generator=gen, device="cuda:0").float()
    A, B = a.to(torch.bfloat16), b.to(torch.bfloat16)
    scratch = torch.empty(8, device="cuda:0")
    want = torch.matmul(a, b.t())  # fp32 sums of 136 whole numbers below 2^24: exact
    for tile in (0, 64, 128, 256):
        C = torch.full((M + 1, N), -1.0, device="cuda:0")
        assert C.numel() * 4 > 256 << 20
        assert _gemm(True, True, A, K, B, K, M, N, K, C, N, tile, 0, scratch) == 0
        assert torch.equal(C[:M], want) and bool((C[M:] == -1.0).all())
