"""GPU eigensolver of the environment, step by step: the isometry a step
applied against the environment it was computed from (both read back through
the C ABI), at the sizes where the kernels' tiling has its edges."""
import numpy as np
import pytest

from paper_2602_05900_amd import workloads

pytestmark = pytest.mark.gpu


def check_pairs(E, U, orth, resid):
    """U's columns orthonormal and eigenvectors of E (Rayleigh quotients), and
    no eigenvalue left out above the kept ones."""
    lam0 = np.linalg.eigvalsh(E)[::-1]
    k = U.shape[1]
    scale = max(abs(lam0[0]), 1e-300)
    th = np.einsum("ij,ij->j", U, E @ U)
    assert np.abs(U.T @ U - np.eye(k)).max() <= orth
    assert np.abs(E @ U - U * th).max() <= resid * scale
    assert np.abs(th - lam0[:k]).max() <= resid * scale


# n = Dx^2 at every block count of the dense solver, its remainders and its
# ends; dy = 1 leaves E of low rank, dy = 4 of full rank
@pytest.mark.parametrize("dx", range(1, 10))
@pytest.mark.parametrize("dy", [1, 4])
def test_dense_environment(gpu_lib, dx, dy):
    from paper_2602_05900_amd import binding
    s = binding.Solve(model="custom", tensor=workloads.random_tensor(dx, dy, seed=10 * dx + dy), dmax=96, max_steps=1)
    s.coarse_grain(1)
    E, U = s.environment(), s.isometry()
    assert U.shape == (dx * dx, dx * dx)
    # a pair stops rotating at 4e-15 of its norms, and later rotations of the last sweep add 8e-15 at most
    # where tried; products over n <= 81 terms round below 81 eps
    check_pairs(E, U, 5e-14, 5e-14)
    s.close()


# block widths 32, 48, 64, 80, 96; n a multiple of 16, odd, and with a partial
# last group of rows
@pytest.mark.parametrize("D", [10, 11, 17, 21, 24, 30, 33, 40, 49])
def test_subspace_environment(gpu_lib, D):
    from paper_2602_05900_amd import binding
    n = 8
    s = binding.Solve(model="ising", temperature=2.3, dmax=D, max_steps=n)
    s.coarse_grain(n)
    assert s.eig_stop(n) == binding.EIG_CONVERGED and s.eig_info(n)[0] > 0
    E, U = s.environment(), s.isometry()
    assert U.shape == (D * D, D)
    # converged pairs: residual at most 1e-12 of the largest eigenvalue; the
    # vectors are products over p <= 96 of columns orthonormal to 96 x 4e-15 (later rotations of the
    # Jacobi's last sweep included: 8e-15 a pair at most where tried, few pairs near it)
    check_pairs(E, U, 4e-13, 1.1e-12)
    s.close()


# deep in the ordered phase most kept pairs lie below 1e-8 of the largest:
# they must not tilt the leading ones
@pytest.mark.parametrize("T", [1.7, 1.8, 1.9])
def test_subspace_steep_spectrum(gpu_lib, T):
    from paper_2602_05900_amd import binding
    s = binding.Solve(model="ising", temperature=T, dmax=48, max_steps=20)
    s.coarse_grain(20)
    s.log_z()
    for n in range(1, 21):
        assert s.eig_info(n)[2] <= 1e-12, (n, s.eig_info(n))
    s.close()


# a pass limit ends the solve on a Ritz pass, which at an odd limit follows no
# power pass: the isometry is orthonormal all the same (to the 4e-13 of the
# converged solves above), and the residual reported is that of unit vectors:
# at least theirs with Rayleigh quotients, which make it smallest
@pytest.mark.parametrize("passes", [1, 2, 3, 5, 7])
@pytest.mark.parametrize("D", [17, 48])
def test_pass_limit_leaves_an_isometry(gpu_lib, passes, D):
    from paper_2602_05900_amd import binding
    n = 8                                     # cold solves at steps 5 and 6, warm ones at 7 and 8
    s = binding.Solve(model="ising", temperature=2.25, dmax=D, max_steps=n)
    s.set_eig_limits(max_passes=passes, fail_residual=1e300)
    for step in range(1, n + 1):
        s.coarse_grain(1)
        E, U = s.environment(), s.isometry()
        assert np.abs(U.T @ U - np.eye(U.shape[1])).max() <= 4e-13
        it, _, resid = s.eig_info(step)
        if it:
            assert it <= passes
            th = np.einsum("ij,ij->j", U, E @ U)
            own = np.sqrt(((E @ U - U * th) ** 2).sum(0)).max()
            assert own <= resid * 1.01 * np.linalg.eigvalsh(E)[-1] + 1e-12 * abs(np.trace(E))
    assert np.isfinite(s.log_z())
    s.close()


# deep in the ordered phase, the columns themselves: a block is factored once as
# it is while its scaled Gram matrix has pivots above 1e-11, which leaves its
# columns orthonormal to p eps / 1e-11 = 1e-3 at worst; the pairs above 1e-7 of
# the largest come first and have pivots near 1, as the converged solves above
@pytest.mark.parametrize("T", [1.7, 1.8, 1.9])
def test_subspace_steep_spectrum_isometry(gpu_lib, T):
    from paper_2602_05900_amd import binding
    s = binding.Solve(model="ising", temperature=T, dmax=48, max_steps=20)
    for _ in range(20):
        s.coarse_grain(1)
        E, U = s.environment(), s.isometry()
        th = np.einsum("ij,ij->j", U, E @ U)
        G = np.abs(U.T @ U - np.eye(U.shape[1]))
        top = th > 1e-7 * th[0]
        assert G.max() <= 1.1e-3
        assert G[np.ix_(top, top)].max() <= 4e-13
    s.close()


# environments of the reduced precisions in the dense solver, n = 4 to 81: they
# are not definite to the first shifts tried.  The isometry is kept in the
# precision's operands, of unit roundoff u: its columns then differ from the
# vectors found by u, E U by u times the largest eigenvalue
@pytest.mark.parametrize("precision,u", [("fp32", 2.0 ** -24), ("bf16x6", 2.0 ** -24), ("bf16x3", 2.0 ** -16)])
@pytest.mark.parametrize("model,q,T,D", [("ising", 2, 1.9, 8), ("ising", 2, 2.3, 9), ("potts", 3, 1.0, 9)])
def test_dense_environment_of_reduced_precision(gpu_lib, precision, u, model, q, T, D):
    from paper_2602_05900_amd import binding
    n, lowest = 12, 0.0
    s = binding.Solve(model=model, q=q, temperature=T, dmax=D, precision=precision, max_steps=n)
    for step in range(1, n + 1):
        s.coarse_grain(1)
        E, U = s.environment(), s.isometry()
        check_pairs(E, U, 5e-14 + 4 * u, 5e-14 + 4 * u)
        assert s.eig_stop(step) == binding.EIG_CONVERGED
        w = np.linalg.eigvalsh(E)
        lowest = min(lowest, w[0] / w[-1])
    if precision == "bf16x3":
        assert lowest < -1e-13        # past the first two shifts
    s.close()
