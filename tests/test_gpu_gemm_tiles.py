"""The matrix product's tile sizes at the edges of tiles, contraction steps and splits, in every operand layout.

Operands are whole numbers of at most 8: every partial sum is a whole number below 2^24, exact in fp32 whatever the
order, so the results have to be equal to the product of the whole numbers, not only close."""
import pytest

pytestmark = pytest.mark.gpu

# (M, N, K): which tile a size takes is decided by its cost; these cover T = 64, 128 and 256, one and several ranges
SIZES = [(8, 8, 8), (8, 1024, 2400), (64, 64, 128), (56, 72, 120), (72, 136, 264), (200, 80, 1000), (624, 400, 1000),
         (1000, 400, 136), (4096, 1024, 512), (4104, 1016, 520), (16384, 264, 72), (2048, 2048, 64), (512, 256, 16384),
         (1032, 520, 8200), (4096, 3200, 1032)]


@pytest.mark.parametrize("a_kc,b_kc", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_product_of_whole_numbers_is_exact(M, N, K, a_kc, b_kc):
    import torch
    from paper_2201_05500_amd import binding_mlp as BM
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M * 31 + N * 7 + K)
    ints = lambda shape: torch.randint(-8, 9, shape, generator=gen, device="cuda:0")
    a, b = ints((M, K)), ints((K, N))
    A = (a if a_kc else a.t()).to(torch.bfloat16).contiguous()
    B = (b.t() if b_kc else b).to(torch.bfloat16).contiguous()
    exact = torch.matmul(a.double(), b.double()).float()
    scratch = torch.empty(8 << 20, dtype=torch.float32, device="cuda:0")
    for scratch_bytes in (scratch.numel() * 4, 0):  # split where that pays, then never split
        # rows behind C tell a store out of range
        C = torch.full((M + 2, N), -1.0, dtype=torch.float32, device="cuda:0")
        st = BM.ctr_mlp_gemm(a_kc, b_kc, A.data_ptr(), A.shape[1], B.data_ptr(), B.shape[1], M, N, K, C.data_ptr(), N,
                             scratch.data_ptr() if scratch_bytes else None, scratch_bytes,
                             torch.cuda.current_stream().cuda_stream)
        assert st == 0
        assert torch.equal(C[:M], exact)
        assert bool((C[M:] == -1.0).all())
