"""GPU test of the device memory a descent holds: the refinement's buffers (two
N x N float64 matrices, N = n rounded up to 32) only where its eigensolves can
refine, counted through the allocator hook."""

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


LAM = 24


def held(alloc):
    assert alloc.live
    return sum(alloc.live.values())


def solo(P, n, precision, variant="standard"):
    with P.CMAES(n, LAM, 1.0, seed=1, precision=precision, variant=variant, objective="sphere", allocator="torch") as es:
        es.generation()
        return held(es.allocator)


def hook(P):
    alloc = P.binding.TorchAllocator()
    return alloc, dict(dev_malloc=alloc.c_malloc, dev_free=alloc.c_free)


def test_concurrent_descents_hold_no_refinement_buffers(P):
    n, two = 160, 2 * 8 * 160 * 160
    print("case memory of concurrent descents", flush=True)
    alone = solo(P, n, "fp64")
    assert alone - solo(P, n, "fp64", "separable") >= two
    R, xs = synth.problem(n, 1)
    alloc, opts = hook(P)
    with P.CMAESBatch([n, n], [LAM, LAM], [1.0, 1.0], [1, 2], precision="fp64", **opts) as b:
        for k in range(2):
            b.set_objective(k, "sphere")
        b.generation()
        assert held(alloc) <= 2 * (alone - two)
    alloc, opts = hook(P)
    r = P.KReplicated(n, LAM, 4, 1.0, seed=1, precision="fp64", objective="sphere", **opts)
    try:
        r.generation()
        assert held(alloc) <= 4 * (alone - two)
    finally:
        r.close()


def test_mixed_descents_hold_refinement_buffers_only_beyond_192(P):
    """From n = 192 to 193 the padded size goes from 192 to 224: about ten float64
    matrices of that size grow, and the two of the refinement come on top."""
    print("case memory of mixed descents", flush=True)
    below, grown = solo(P, 192, "mixed"), solo(P, 193, "mixed")
    steady = solo(P, 160, "mixed")
    assert (grown - below) - (below - steady) >= 8 * 224 * 224
    assert solo(P, 64, "fp64") < solo(P, 65, "fp64") - 2 * 8 * 96 * 96
