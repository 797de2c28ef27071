"""GPU test of the per-kernel times (cmaes_kernel_times): every float64 product of a
refining eigensolve is counted, the triangular ones among them."""

import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_11765_amd as P
    return P


@pytest.mark.parametrize("n", [100, 400, 700])
def test_every_product_of_the_refinement_is_timed(P, n):
    """Two products start a solve; its first step takes at least two (Theta^2, V X),
    each later one at least four (C V, S with G, Theta^2, V X)."""
    print(f"case kernel times n={n}", flush=True)
    lam = 3 * n
    with P.CMAES(n, lam, 1.0, seed=3, precision="fp64", objective="sphere", eigen_interval=1) as es:
        es.set_state(synth.random_state(n, lam, seed=n, cond=30.0))
        es.enable_kernel_timing(True)
        es.generation()
        s = es.state(arrays=False)
        t = es.kernel_times()["eig_gemm"]
    steps = s["eig_sweeps"] + s["eig_corrections"]
    assert steps >= 2
    assert t["calls"] >= 4 * steps and t["total_us"] > 0.0, (t, steps)
