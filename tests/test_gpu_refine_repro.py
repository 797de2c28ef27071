"""GPU tests of the refinement's reproducibility (C = B D^2 B^T, Sec. 2.1): what a
solve computes follows from the state that it starts from, not from how fast the
host queues its steps nor from what the solve before it happened to need."""

import numpy as np
import pytest

import synth
from test_gpu_eigen_correction import check_decomposition

pytestmark = pytest.mark.gpu

ARRAYS = ("m", "C", "B", "D", "p_sigma", "p_c", "f", "order")


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_11765_amd as P
    return P


def same(a, b, what):
    for k in ARRAYS:
        assert np.array_equal(a[k], b[k]), (what, k)
    assert (a["sigma"], a["eig_sweeps"], a["eig_corrections"]) == (b["sigma"], b["eig_sweeps"], b["eig_corrections"]), what


@pytest.mark.parametrize("n,lam", [(130, 24), (200, 400), (400, 24)])
def test_first_generations_are_reproducible(P, n, lam):
    """From C = I, where solves sweep, take single steps and queue many at once:
    two runs of one seed, and graphs on against off, bit for bit.  The timing
    differs between them, the results may not."""
    print(f"case reproducible n={n} lam={lam}", flush=True)
    R, xs = synth.problem(n, n)

    def run(graphs):
        with P.CMAES(n, lam, 2.0, seed=11, precision="fp64", objective="rastrigin", R=R, xstar=xs, f_target=0.0,
                     eigen_interval=1) as es:
            es.enable_graphs(graphs)
            for _ in range(20):
                es.generation()
                yield es.state()

    for g, (a, b, c) in enumerate(zip(run(True), run(True), run(False))):
        same(a, b, (g, "twice"))
        same(a, c, (g, "eager"))


def handle(P, n, lam):
    return P.CMAES(n, lam, 1.0, seed=3, precision="fp64", objective="sphere", f_target=0.0, eigen_interval=1)


@pytest.mark.parametrize("n", [100, 200, 400])
def test_resumed_descent_equals_the_one_that_ran_on(P, n):
    """A descent whose state goes out and back in before every generation: the solve
    after that knows nothing of the solves before it, and must still do as they do."""
    print(f"case resumed n={n}", flush=True)
    lam = 3 * n
    st = synth.random_state(n, lam, seed=n, cond=30.0)
    with handle(P, n, lam) as on, handle(P, n, lam) as resumed:
        on.set_state(st)
        resumed.set_state(st)
        for g in range(8):
            on.generation()
            resumed.set_state(resumed.state())
            resumed.generation()
            same(on.state(), resumed.state(), g)


def turned(n, seed, size):
    """A rotation by angles whose squares sum to size^2 in each row, on average."""
    K = synth.rng(seed).standard_normal((n, n))
    q, r = np.linalg.qr(np.eye(n) + size * (K - K.T) / np.sqrt(2 * n))
    return q * np.sign(np.diag(r))


@pytest.mark.parametrize("n", [96, 385, 700])
@pytest.mark.parametrize("what", ["C", "p_c"])
def test_large_angles_after_solves_with_none(P, n, what):
    """A steady descent, then C replaced without B, or the evolution path, which
    moves C far along one direction: the next solve's first step has long rows and
    large angles that none of the solves before it had, and must treat them as a
    solve of the same state on a new handle does."""
    print(f"case large angles after none n={n} {what}", flush=True)
    lam = 3 * n
    with handle(P, n, lam) as es, handle(P, n, lam) as new:
        es.set_state(synth.random_state(n, lam, seed=n, cond=30.0))
        for _ in range(4):
            es.generation()
        s = es.state()
        part = {"n": n, "lambda": lam, "gen": s["gen"], "sigma": s["sigma"]}
        if what == "C":
            Q = turned(n, n + 1, 1.0)
            C = Q @ s["C"] @ Q.T
            part["C"] = 0.5 * (C + C.T)
        else:
            part["p_c"] = 30.0 * n * synth.rng(n + 2).standard_normal(n)
        es.set_state(part)
        new.set_state({**s, **part})
        es.generation()
        new.generation()
        a, b = es.state(), new.state()
        check_decomposition(a)
        same(a, b, what)
