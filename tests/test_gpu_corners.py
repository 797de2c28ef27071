"""GPU tests of two corners: the active covariance update (two operands) in every
tile of the float64 product at sizes whose leading dimension is not n, and eigensolves
whose refinement is given up for good."""

import numpy as np
import pytest

import synth
from helpers import FTOL, RANK_TAU, TOL, rank_agreement, rel
from test_gpu_refine import P  # noqa: F401 (the fixture)
from test_gpu_variants import _one_generation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lam", [(851, 1537), (851, 400), (853, 190)])
def test_active_update_in_every_tile(P, n, lam):  # noqa: F811
    """Tiles of 48, the product split over k, tiles of 16."""
    print(f"case active update n={n} lam={lam}", flush=True)
    g, o, info, _ = _one_generation(P, "active", "fp64", n, lam, "ellipsoid", False)
    assert np.max(np.abs(g["f"] - info["f"]) / np.abs(info["f"])) <= FTOL["fp64"]
    assert rank_agreement(info["f"], g["order"], info["order"], RANK_TAU["fp64"]) == 0
    for k, a, b in (("m", g["m"], o.m), ("C", g["C"], o.C), ("p_c", g["p_c"], o.pc), ("p_sigma", g["p_sigma"], o.ps)):
        assert rel(a, b) < TOL["fp64"], k
    assert np.array_equal(g["C"], g["C"].T)


@pytest.mark.parametrize("n", [65, 200, 400])
def test_refinement_given_up(P, n):  # noqa: F811
    """B one and a half times an orthogonal matrix: every step finds it too far from
    orthogonal, and the solve starts over with sweeps alone.  They turn B by rotations,
    so it keeps its length, as in a solve that is told not to refine."""
    print(f"case refinement given up n={n}", flush=True)
    lam = 2 * n
    st = synth.random_state(n, lam, seed=n, cond=30.0)
    st["B"] = 1.5 * st["B"]
    out = []
    for on in (True, False):
        with P.CMAES(n, lam, 1.0, seed=3, precision="fp64", objective="sphere", eigen_interval=1) as es:
            es.set_eigen_correction(on)
            es.set_state(st)
            es.generation()
            out.append(es.state())
    a, b = out
    assert np.array_equal(a["C"], b["C"])
    for s in out:
        B, D2 = s["B"] / 1.5, s["D"] ** 2 / 2.25
        assert np.max(np.abs(B.T @ B - np.eye(n))) <= 1e-12
        assert rel((B * D2) @ B.T, s["C"]) <= 1e-12
    assert rel(a["D"], b["D"]) <= 1e-12
    assert a["eig_sweeps"] >= 3
