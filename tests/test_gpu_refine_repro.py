"""GPU tests of the refinement's reproducibility (C = B D^2 B^T, Sec. 2.1): what a
solve computes follows from the state that it starts from, not from how fast the
host queues its steps nor from what the solve before it happened to need."""

import numpy as np
import pytest

import synth

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
