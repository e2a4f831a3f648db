"""The product kernel at the edges of its tile choices (binding.gemm_nt)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UNIT = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "bf16x6": 2.0 ** -24, "bf16x3": 2.0 ** -16}


def check_product(M, N, K, precision, role="generic"):
    """C = A B^T within (2 + 8 sqrt K) u sum_k |a_k b_k|, u the unit roundoff
    of the arithmetic (operands of odd leading dimensions)."""
    import torch
    from paper_2602_05900_amd import binding
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    lda, ldb = K + 2, K + 1
    A, B = rng.standard_normal((M, lda)), rng.standard_normal((N, ldb))
    C = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    binding.gemm_nt(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), C, M, N, K, lda, ldb, (1, N, 0, N, 0, 1),
                    precision=precision, role=role)
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
