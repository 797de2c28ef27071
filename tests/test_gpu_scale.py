"""GPU tests of the eigensolve (C = B D^2 B^T, Sec. 2.1) at the ends of float64's
range: a covariance whose entries' squares overflow is refused as non-finite, one
whose entries' squares underflow is decomposed as any other."""

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


def scaled(n, lam, exponent):
    """A descent's state with C times 4^exponent."""
    st = synth.random_state(n, lam, seed=n, cond=100.0)
    s = 2.0 ** exponent
    return {**st, "C": st["C"] * s * s, "D": st["D"] * s, "p_c": st["p_c"] * s}


@pytest.mark.parametrize("n", [10, 40, 64, 100])
def test_overflowing_covariance_is_refused(P, n):
    print(f"case overflow n={n}", flush=True)
    lam = 3 * n
    with P.CMAES(n, lam, 1.0, seed=3, precision="fp64", objective="sphere", eigen_interval=1) as es:
        es.set_state(scaled(n, lam, 270))
        assert P.library().cmaes_generation(es.h) == P.binding.CMAES_ENUMERIC
        assert "conditioncov" in es.state(arrays=False)["stop_names"]


@pytest.mark.parametrize("n", [10, 31, 40, 64])
def test_underflowing_covariance_is_decomposed(P, n):
    print(f"case underflow n={n}", flush=True)
    lam, e = 3 * n, -300
    with P.CMAES(n, lam, 1.0, seed=3, precision="fp64", objective="sphere", eigen_interval=1) as es:
        es.set_state(scaled(n, lam, e))
        es.generation()
        s = es.state()
    check_decomposition({"C": s["C"] * 4.0 ** -e, "B": s["B"], "D": s["D"] * 2.0 ** -e})
    assert "conditioncov" not in s["stop_names"]
