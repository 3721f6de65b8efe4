"""The matrix product's tile sizes at the edges of tiles, contraction steps and splits, in every operand layout.

Operands are whole numbers of at most 8: every partial sum is a whole number below 2^24, exact in fp32 whatever the
order, so the results have to be equal to the product of the whole numbers, not only close."""
import pytest

pytestmark = pytest.mark.gpu

# (M, N, K): which tile a size takes is decided by its cost; tests/test_gemm_plan.py says which these take
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


# (M, N, K): tests/test_gemm_plan.py has the ranges of each: one, many of 256, many whose length is an odd number of 64s
# (a step of the 64-wide tile, 128, then reaches beyond a range's end in mid-contraction), a last one that ends in mid-step; the
# most ranges whose partial sums a small product adds eight at a time, and one more
BITS = [(72, 136, 264), (640, 96, 640), (264, 200, 1288), (136, 72, 9224), (1000, 400, 5768), (1032, 520, 5768),
        (1032, 520, 8200), (16, 200, 2160), (16, 200, 2560)]


@pytest.mark.parametrize("a_kc,b_kc", [(True, False), (False, False), (True, True), (False, True)])
@pytest.mark.parametrize("M,N,K", BITS)
def test_product_has_the_same_bits_whatever_the_tile_and_the_split(M, N, K, a_kc, b_kc):
    import torch
    from paper_2201_05500_amd import binding_mlp as BM
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M + N + K)
    a = torch.randn((M, K), generator=gen, device="cuda:0").to(torch.bfloat16)
    b = torch.randn((K, N), generator=gen, device="cuda:0").to(torch.bfloat16)
    A = (a if a_kc else a.t()).contiguous()
    B = (b.t() if b_kc else b).contiguous()
    exact, weight = torch.matmul(a.double(), b.double()), torch.matmul(a.double().abs(), b.double().abs())
    scratch = torch.empty(8 << 20, dtype=torch.float32, device="cuda:0")
    ran = 0
    for room in (scratch.numel() * 4, 0):  # without room there is one range
        first = None
        ranges = BM.ctr_debug_mlp_gemm_plan(M, N, K, room)[2]
        for tile, split in ((64, 0), (64, 1), (128, 0), (128, 1), (256, 0), (256, 1), (0, 0)):
            C = torch.full((M + 2, N), -1.0, dtype=torch.float32, device="cuda:0")
            st = BM.ctr_debug_mlp_gemm(a_kc, b_kc, A.data_ptr(), A.shape[1], B.data_ptr(), B.shape[1], M, N, K,
                                       C.data_ptr(), N, scratch.data_ptr() if room else None, room, tile, split,
                                       torch.cuda.current_stream().cuda_stream)
            if tile == 256 and not split and ranges > 1:
                assert st != 0  # the large tile takes one range per work item
                continue
            assert st == 0 and bool((C[M:] == -1.0).all()), (tile, split)
            ran += 1
            if first is None:
                first = C[:M].clone()
                # fp32 sums of K exact products: at most K roundings of a partial sum, each within 2^-24 of the sum of
                # the magnitudes
                assert bool(((first.double() - exact).abs() <= K * 2.0 ** -24 * weight).all())
            assert torch.equal(C[:M], first), (tile, split, room)
    assert ran >= 12
    assert BM.ctr_debug_mlp_gemm(a_kc, b_kc, A.data_ptr(), A.shape[1], B.data_ptr(), B.shape[1], M, N, K, C.data_ptr(), N,
                                 None, 0, 32, 0, torch.cuda.current_stream().cuda_stream) != 0
