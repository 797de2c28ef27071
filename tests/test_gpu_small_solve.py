"""GPU tests of the eigensolve of up to 64 dimensions in one workgroup
(C = B D^2 B^T, Sec. 2.1): sizes at the edges of its 16 x 16 blocks and of its
two kernels (32, 64), odd sizes (a rotation round then has an idle player), and
starts that take each of its paths (steps at once; sweeps first; sweeps between
steps; a start over from the identity).  The decomposition must meet the bar of
every other solve: C = B D^2 B^T, B^T B = I and the eigenvalues of a library
eigensolver to 1e-12."""

import numpy as np
import pytest

import synth
from test_gpu_eigen_correction import check_decomposition
from test_gpu_refine import P, decompose  # noqa: F401 (P: the fixture)

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64]


@pytest.mark.parametrize("n", SIZES)
def test_small_solve_from_near_and_from_afar(P, n):  # noqa: F811
    """B the eigenvectors of C before its update, then unrelated to it."""
    print(f"case small solve n={n}", flush=True)
    lam = 3 * n + 4
    st = synth.random_state(n, lam, seed=n, cond=100.0)
    check_decomposition(decompose(P, st, lam, gens=2))
    st["B"] = synth.haar_rotation(n, n + 7)
    check_decomposition(decompose(P, st, lam))


@pytest.mark.parametrize("n,rank", [(16, 1), (33, 3), (64, 7)])
def test_small_solve_of_multiple_eigenvalues(P, n, rank):  # noqa: F811
    """C = I plus a low rank: angles that add up, so sweeps come between the steps."""
    print(f"case small solve multiple eigenvalue n={n} rank={rank}", flush=True)
    st = synth.random_state(n, 8, seed=n, cond=1.0)
    Y = synth.rng(n).standard_normal((n, rank))
    st["C"] = np.eye(n) + Y @ Y.T / n
    st["B"], st["D"] = np.eye(n), np.ones(n)
    check_decomposition(decompose(P, st, 8, gens=5))


@pytest.mark.parametrize("n", [17, 64])
def test_small_solve_of_a_wide_spectrum(P, n):  # noqa: F811
    """Eigenvalues over ten decades: the small ones lie below the products' rounding."""
    print(f"case small solve wide spectrum n={n}", flush=True)
    st = synth.random_state(n, 2 * n, seed=n, cond=1e10)
    check_decomposition(decompose(P, st, 2 * n, gens=2))


@pytest.mark.parametrize("n", [31, 64])
def test_small_solve_starts_over_from_the_identity(P, n):  # noqa: F811
    """B far from orthogonal (two columns alike): no basis to start from."""
    print(f"case small solve without a basis n={n}", flush=True)
    st = synth.random_state(n, 2 * n, seed=n, cond=50.0)
    st["B"][:, 1] = st["B"][:, 0]
    check_decomposition(decompose(P, st, 2 * n))


def test_small_solves_of_both_sizes_in_one_group(P):  # noqa: F811
    """Concurrent descents on both sides of 32 dimensions, and one beyond 64."""
    print("case small solves in a group", flush=True)
    ns, lams = [20, 33, 64, 32, 70], [12, 24, 40, 16, 20]
    with P.CMAESBatch(ns, lams, [1.0] * 5, list(range(5)), precision="fp64") as b:
        for k in range(5):
            b.set_objective(k, "sphere")
        for _ in range(6):
            b.generation()
        for k in range(5):
            s = b.state(k)
            if s["gen"] % s["kappa"] == 0:   # the decomposition ran in this generation
                check_decomposition(s)
