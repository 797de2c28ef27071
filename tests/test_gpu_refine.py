"""GPU tests of the eigensolve's refinement by products (C = B D^2 B^T, Sec. 2.1).

One generation from an injected state whose B is exactly, nearly or not at all
the eigenvectors of the covariance that the generation produces: the solve then
refines at once, over several steps, or only after sweeps.  Sizes sit at the
edges of the product tiles (16, 32 and 48), of the padding to 32 and of the
ranges the tiles are chosen by (384, 640).  The decomposition must meet the bar
of a sweeps-only solve: C = B D^2 B^T, B^T B = I and the eigenvalues of a
library eigensolver to 1e-12."""

import numpy as np
import pytest

import synth
from test_gpu_eigen_correction import check_decomposition

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_11765_amd as P
    return P


def decompose(P, st, lam, gens=1):
    n = st["n"]
    with P.CMAES(n, lam, 1.0, seed=3, precision="fp64", objective="sphere", eigen_interval=1) as es:
        es.set_state(st)
        for _ in range(gens):
            es.generation()
        return es.state()


@pytest.mark.parametrize("n", [65, 80, 96, 97, 113, 160, 191, 383, 384, 385, 639, 640, 641, 673])
def test_refinement_at_tile_edges(P, n):
    """Separated eigenvalues and a population of 3 n: nearly diagonal from the start."""
    print(f"case refine n={n}", flush=True)
    lam = 3 * n
    s = decompose(P, synth.random_state(n, lam, seed=n, cond=100.0), lam)
    check_decomposition(s)
    assert s["eig_corrections"] >= 1    # the last step's angles are small


@pytest.mark.parametrize("n", [100, 200, 500, 700])
def test_refinement_after_sweeps(P, n):
    """B unrelated to C: angles of every size, swept before they are refined."""
    print(f"case refine from an unrelated basis n={n}", flush=True)
    st = synth.random_state(n, 2 * n, seed=n, cond=30.0)
    st["B"] = synth.haar_rotation(n, n + 7)
    check_decomposition(decompose(P, st, 2 * n))


@pytest.mark.parametrize("n,rank", [(100, 7), (300, 40), (700, 3)])
def test_refinement_of_multiple_eigenvalues(P, n, rank):
    """C = I plus a low rank: inside the multiple eigenvalue the basis is
    arbitrary and angles are rounding divided by rounding."""
    print(f"case refine multiple eigenvalue n={n} rank={rank}", flush=True)
    st = synth.random_state(n, 8, seed=n, cond=1.0)
    g = synth.rng(n)
    Y = g.standard_normal((n, rank))
    st["C"] = np.eye(n) + Y @ Y.T / n
    st["B"], st["D"] = np.eye(n), np.ones(n)
    check_decomposition(decompose(P, st, 8, gens=3))


@pytest.mark.parametrize("n", [96, 400])
def test_refinement_of_a_wide_spectrum(P, n):
    """Eigenvalues over ten decades: the small ones lie below the products' rounding."""
    print(f"case refine wide spectrum n={n}", flush=True)
    st = synth.random_state(n, 2 * n, seed=n, cond=1e10)
    check_decomposition(decompose(P, st, 2 * n, gens=2))


def test_refinement_removes_the_drift_of_an_inexact_basis(P):
    """B given orthogonal to 1e-6 only: the steps take its distance from
    orthogonality out with the off-diagonal part."""
    n, lam = 200, 400
    st = synth.random_state(n, lam, seed=5, cond=100.0)
    st["B"] = st["B"] + 1e-8 * synth.rng(9).standard_normal((n, n))
    check_decomposition(decompose(P, st, lam))


@pytest.mark.parametrize("n,lam", [(100, 17), (400, 24)])
def test_refinement_from_the_identity(P, n, lam):
    """The first generations of a search, C = I plus ever more outer products:
    steps are refused, go astray and are recovered from, and wait their turn."""
    print(f"case refine from the identity n={n}", flush=True)
    R, xstar = synth.problem(n, 1)
    with P.CMAES(n, lam, 2.0, seed=5, precision="fp64", objective="rastrigin", R=R, xstar=xstar, f_target=0.0,
                 eigen_interval=1) as es:
        for _ in range(14):
            es.generation()
            check_decomposition(es.state())


@pytest.mark.parametrize("n", [65, 96, 130, 383, 385, 641])
def test_refinement_damps_long_rows(P, n):
    """B turned away from C's eigenvectors by angles whose rows are longer than a
    step takes: their tiles are scaled, in both triangles, before they are applied."""
    print(f"case refine with long rows n={n}", flush=True)
    st = synth.random_state(n, 2 * n, seed=n, cond=30.0)
    K = synth.rng(n + 1).standard_normal((n, n))
    q, r = np.linalg.qr(np.eye(n) + 0.5 * (K - K.T) / np.sqrt(n))
    st["B"] = st["B"] @ (q * np.sign(np.diag(r)))
    check_decomposition(decompose(P, st, 2 * n))
