"""GPU tests of the launches between sampling and the covariance update, at the
sizes where they change: 32 rows to a workgroup; products of up to 512 columns in
one launch, larger ones in chunks; sums over up to 8192 / n chunks of 64 ranks on
the way; 256 keys to a sorted chunk, 8 chunks to a merge; the objective's shift
beside the normals up to 1024 of their workgroups; float64 products in tiles of
16 and 32, covariance updates in tiles of 16 and 48 or split.  One generation against the
float64 oracle, to the bars of the parity tests."""

import numpy as np
import pytest

import oracle as O
import synth
from helpers import one_generation, oracle_state, rel
from test_gpu_parity import P, check_one_generation  # noqa: F401 (P: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,lam", [(31, 2), (32, 128), (33, 130), (64, 256), (65, 257), (512, 2048), (512, 2176),
                                   (513, 512), (20, 2049), (40, 4100), (15, 17), (16, 16), (129, 1041), (127, 96), (851, 301), (851, 3090)])
def test_one_generation_at_the_edges(P, precision, n, lam):  # noqa: F811
    print(f"case front {precision} n={n} lam={lam}", flush=True)
    st = synth.random_state(n, lam, seed=n * 5 + lam, cond=50.0)
    R, xs = synth.problem(n, seed=n + 2)
    Z = synth.normal_matrix(n, lam, seed=lam * 13 + n)
    g, o, info = one_generation(P, st, Z, "ellipsoid", R, xs, precision)
    if precision == "mixed":
        # float32 values this close swap neighbouring ranks: the oracle goes on
        # from the device's values, whose order it must find
        f_ref = info["f"]
        o = oracle_state(st)
        info = O.generation(o, O.Objective("ellipsoid", R, xs), Z=Z, fvals=g["f"])
        assert np.array_equal(g["order"], info["order"])
        info["f"] = f_ref
    check_one_generation(g, o, {**info, "order": O.rank_order(info["f"])}, precision, st, lam)
    best = int(g["order"][0])
    assert g["f_best"] == g["f"][best]
    X = st["m"] + st["sigma"] * (st["B"] @ (st["D"] * Z[:, best]))
    assert rel(g["x_best"], X) < (1e-12 if precision == "fp64" else 1e-5)


@pytest.mark.parametrize("n,lam,rotated", [(32, 40, True), (33, 40, False), (300, 60, False), (400, 2600, True),
                                           (400, 2700, True), (512, 64, True), (513, 64, True)])
def test_shift_beside_the_normals(P, n, lam, rotated):  # noqa: F811
    """The fused launch and a caller's own normals (the same ones) agree."""
    print(f"case shift n={n} lam={lam} rotated={rotated}", flush=True)
    st = synth.random_state(n, lam, seed=n + lam, cond=50.0)
    R, xs = synth.problem(n, seed=n + 2) if rotated else (None, synth.optimum(n, n + 2))
    out = []
    for given in (False, True):
        with P.CMAES(n, lam, 1.0, seed=9, precision="fp64", objective="rastrigin", R=R, xstar=xs) as es:
            es.set_state(st)
            if given:
                es.generation_with_z(O.normals(9, 0, st["gen"], n, lam))
            else:
                es.generation()
            out.append(es.state())
    assert np.array_equal(out[0]["order"], out[1]["order"])
    assert rel(out[0]["f"], out[1]["f"]) < 1e-11
    for k in ("m", "p_sigma", "p_c"):
        assert rel(out[0][k], out[1][k]) < 1e-12, k
