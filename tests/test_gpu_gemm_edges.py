"""The product kernel at the edges of its tile choices (binding.gemm_nt)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UNIT = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "bf16x6": 2.0 ** -24, "bf16x3": 2.0 ** -16}


def check_product(M, N, K, precision, role="generic", pad=(2, 1), panel=False):
    """C = A B^T within (2 + 8 sqrt K) u sum_k |a_k b_k|, u the unit roundoff
    of the arithmetic (operands of leading dimensions K + pad)."""
    import torch
    from paper_2602_05900_amd import binding
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    lda, ldb = K + pad[0], K + pad[1]
    A, B = rng.standard_normal((M, lda)), rng.standard_normal((N, ldb))
    C = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    binding.gemm_nt(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), C, M, N, K, lda, ldb, (1, N, 0, N, 0, 1),
                    precision=precision, role=role, panel=panel)
    ref = A[:, :K] @ B[:, :K].T
    bound = (2.0 + 8.0 * np.sqrt(K)) * UNIT[precision] * (np.abs(A[:, :K]) @ np.abs(B[:, :K]).T) + 1e-300
    assert np.all(np.abs(C.cpu().numpy() - ref) <= bound)


# K not a multiple of 16, split precisions: 64 x 64 tiles, 128 x 128 and
# 256 x 64 from 256 such tiles up (256 x 256: 16 x 16 of them), one short of
# and one past each edge
@pytest.mark.parametrize("M,N,K", [(63, 65, 21), (64, 64, 1), (129, 441, 7), (1921, 2048, 17), (2049, 2048, 17),
                                   (4096, 3841, 9), (3840, 3841, 9), (65281, 30, 15), (65280, 64, 15), (441, 21, 441)])
@pytest.mark.parametrize("precision", ["bf16x3", "bf16x6"])
def test_ragged_k_tiles(gpu_lib, M, N, K, precision):
    check_product(M, N, K, precision)


# FP64: K split over the waves of 32 x 32 tiles up to 256 tiles of 64 x 64 and
# from K = 32: ragged in M, N and K (rows of odd length), fewer groups of 16
# k than waves, and one past either end of the rule
@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (31, 33, 33), (64, 64, 64), (32, 32, 128), (33, 65, 1025), (512, 32, 1024),
                                   (576, 576, 576), (1024, 1024, 47), (1025, 1024, 64), (100, 70, 31), (13824, 24, 576)])
@pytest.mark.parametrize("role", ["generic", "y", "tp"])
def test_fp64_split_k(gpu_lib, M, N, K, role):
    check_product(M, N, K, "fp64", role)


# FP64 with even K and rows (operand tiles loaded straight into LDS): each tile
# of the rule at ragged M and N, stages left over in K, a partial last stage
@pytest.mark.parametrize("M,N,K", [
    (1, 1, 2), (65, 33, 16), (500, 700, 30),                    # 64 x 32: short K
    (576, 576, 98), (8200, 31, 64), (16401, 32, 18),            # 64 x 32: few tiles, narrow
    (1100, 1030, 62), (50, 9000, 50), (9001, 63, 34),           # 64 x 64
    (13050, 700, 34), (129, 65601, 16),                         # 128 x 64
    (13217, 630, 48), (13217, 640, 66), (13217, 638, 2)])       # 128 x 128
@pytest.mark.parametrize("pad", [(0, 0), (4, 2)])
def test_fp64_direct_to_lds(gpu_lib, M, N, K, pad):
    check_product(M, N, K, "fp64", pad=pad)


# the same products with an odd row length or K: staged through registers
@pytest.mark.parametrize("M,N,K", [(1100, 1030, 62), (1100, 1030, 61), (16500, 1030, 17)])
def test_fp64_odd_rows(gpu_lib, M, N, K):
    check_product(M, N, K, "fp64")


# ragged K in the split precisions, few tiles: partial ones, a few K steps and
# many, a partial last step, 192 tiles of 64 x 64 and one row more
@pytest.mark.parametrize("M,N,K", [(1, 1, 33), (31, 33, 47), (32, 64, 127), (33, 65, 129), (441, 441, 441), (100, 70, 1025),
                                   (768, 1024, 63), (769, 1024, 63), (12288, 21, 41)])
@pytest.mark.parametrize("precision", ["bf16x3", "bf16x6"])
@pytest.mark.parametrize("role", ["generic", "x"])
def test_ragged_k_split(gpu_lib, M, N, K, precision, role):
    check_product(M, N, K, precision, role)


# operands converted to whole 32 x 16 panels: one panel, several each way, rows
# of odd length
@pytest.mark.parametrize("M,N,K", [(32, 96, 16), (96, 160, 48), (32, 2048, 16), (1056, 96, 80)])
@pytest.mark.parametrize("precision", ["bf16x3", "bf16x6"])
def test_panel_operands(gpu_lib, M, N, K, precision):
    check_product(M, N, K, precision, role="y", panel=True)


# FP32, few tiles: partial ones, a few K steps and many, 256 tiles of 64 x 64 and
# one row more
@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (31, 33, 33), (33, 65, 1025), (576, 576, 576), (100, 70, 31),
                                   (1024, 1024, 47), (1025, 1024, 64), (16384, 24, 100)])
def test_fp32_split_k(gpu_lib, M, N, K):
    check_product(M, N, K, "fp32")


def check_bits(M, N, K, wide, precision, role="generic"):
    """The M x N product, few tiles, against the first M rows of the product
    with `wide` rows, many tiles of a larger size: the same bits, since K is
    summed in one order whatever the tile."""
    import torch
    from paper_2602_05900_amd import binding
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    A = torch.randn(wide, K, dtype=torch.float64, device="cuda", generator=g)
    B = torch.randn(N, K, dtype=torch.float64, device="cuda", generator=g)
    small = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    large = torch.full((wide, N), float("nan"), dtype=torch.float64, device="cuda")
    for C, rows in ((small, M), (large, wide)):
        binding.gemm_nt(A, B, C, rows, N, K, K, K, (1, N, 0, N, 0, 1), precision=precision, role=role)
    assert torch.equal(small, large[:M])


# 64 x 64 tiles (the small product) and 256 x 128 (1024 tiles of 128 x 128)
@pytest.mark.parametrize("M,N,K", [(1, 129, 32), (64, 257, 441), (577, 300, 576), (1024, 1024, 47)])
def test_fp32_bits_whatever_the_tile(gpu_lib, M, N, K):
    check_bits(M, N, K, 128 * -(-1024 // -(-N // 128)), "fp32")


# ragged K in the split precisions: 64 x 64 or 128 x 128 tiles, and 256 x 256
# (256 x 64 for N <= 64) at 256 of them
@pytest.mark.parametrize("M,N,K", [(1, 129, 33), (64, 257, 441), (577, 300, 577), (2100, 2048, 47), (441, 21, 441)])
@pytest.mark.parametrize("precision", ["bf16x3", "bf16x6"])
@pytest.mark.parametrize("role", ["generic", "y"])
def test_ragged_k_bits_whatever_the_tile(gpu_lib, M, N, K, precision, role):
    check_bits(M, N, K, 256 * 256 if N <= 64 else 256 * -(-256 // -(-N // 256)), precision, role)
