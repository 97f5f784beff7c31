"""The whole-cell step of the fused path at the edges of its range: sets with
points that have no mirror (in whole waves), an odd set, a first stage kept in
LDS in part, one wave per cell, the blocked form of a mesh with few cells, and
a call that fails in the middle.  Bounds are the parity tests' (1e-12 on the
state, 1e-5 for the FP32 form)."""

import numpy as np
import pytest

import ugks_cases as uc
from paper_2606_15720_amd.ugks import UGKS_ENUMERIC, UGKS_FP32, Batch, Solver, UGKSError
from test_gpu_parity import _compare_step, _normwise

pytestmark = pytest.mark.gpu


def _tets(n, vel, K=0):
    case = uc.sod3d_tets(n=n, nv=4, jitter=0.15, seed=3)
    case.vel = vel
    case.gas.K = K
    left = case.mesh.cell_centroid[:, 0] < 0.5
    case.W0 = uc.uniform_W(case.mesh.n_cells, 3, np.where(left, 1.0, 0.6), (0.05, 0.0, 0.0),
                           np.where(left, 1.0, 0.9), K=K)
    return case


def _case(which):
    if which == "sparse_3d":  # 960 points, 288 without a mirror: 336 pairs and 4 waves of single points
        return _tets(2, uc.locally_refined_grid(8, 4.0, 3, (1.2, 0.0, 0.0), 1.8))
    if which == "sparse_3d_internal":
        return _tets(2, uc.locally_refined_grid(8, 4.0, 3, (1.2, 0.0, 0.0), 1.8), K=2)
    if which == "sparse_2d":  # 346 points, 110 without a mirror
        return uc.cavity2d(n=7, kn=0.05, velocity=uc.locally_refined_grid(16, 4.0, 2, (1.1, 0.3), 1.4))
    if which == "odd":  # 15^3: the zero velocity is its own mirror
        return _tets(2, uc.midpoint_grid(15, 4.0, 3))
    if which == "kept_partly":  # 8,788 pairs, of which LDS keeps some 4,000 (FP64)
        return _tets(2, uc.midpoint_grid(26, 4.0, 3))
    if which == "one_wave":  # 4,900 cells of 32 pairs
        return uc.cavity2d(n=70, nv=8, kn=0.05)
    assert which == "blocked"  # 6 cells, 2,916 pairs: two blocks of velocities
    return _tets(1, uc.midpoint_grid(18, 4.0, 3))


EDGES = ["sparse_3d", "sparse_3d_internal", "sparse_2d", "odd", "kept_partly", "one_wave", "blocked"]


@pytest.mark.parametrize("limiter", [0, 1])
@pytest.mark.parametrize("which", EDGES)
def test_whole_cell_edges_follow_the_oracle(which, limiter):
    _compare_step(_case(which), 3, limiter=limiter, limiter_k=0.5)


@pytest.mark.parametrize("limiter", [0, 1])
@pytest.mark.parametrize("which", EDGES)
def test_whole_cell_edges_fp32_form(which, limiter):
    a = Solver(_case(which), limiter=limiter, limiter_k=0.5)
    b = Solver(_case(which), limiter=limiter, limiter_k=0.5, precision=UGKS_FP32)
    a.step(4)
    b.step(4)
    err = _normwise(b.W(), a.W())
    print(which, "FP32 form normwise error:", err, flush=True)
    assert np.all(err < 1e-5)
    a.close()
    b.close()


def _unstable(cfl):
    case = uc.cavity2d(n=8, nv=8, kn=0.05, lid=0.4)
    case.gas.cfl = cfl
    return case


@pytest.mark.parametrize("cfl", [3.5, 4.0, 5.0, 6.0])
def test_a_call_that_fails_in_the_middle_keeps_the_step_before(cfl):
    a = Solver(_unstable(cfl))
    kept, good = a.state(), 0
    for _ in range(100):
        try:
            a.step(1)
        except UGKSError as e:
            assert e.code == UGKS_ENUMERIC
            break
        kept, good = a.state(), good + 1
    else:
        pytest.fail("the case did not fail")
    print("cfl", cfl, "steps before the failure:", good, flush=True)
    for more in (1, 2, 3):
        b = Solver(_unstable(cfl))
        with pytest.raises(UGKSError) as e:
            b.step(good + more)
        assert e.value.code == UGKS_ENUMERIC
        for x, y in zip(b.state(), kept):
            np.testing.assert_array_equal(x, y)
        b.close()
    a.close()
    # in a batch the other case goes on
    fine = uc.cavity2d(n=6, nv=8)
    c, d = Batch([fine, _unstable(cfl)]), Batch([fine])
    d.step(good + 2)
    with pytest.raises(UGKSError) as e:
        c.step(good + 2)
    assert e.value.code == UGKS_ENUMERIC
    np.testing.assert_array_equal(c.W(0), d.W(0))
    # (rounding grows with the unstable mode, from 1e-16; a step more or less is over 1e-3 away)
    assert np.all(_normwise(c.W(1), kept[0]) <= 1e-8)
    c.close()
    d.close()


def test_residual_of_a_call_is_its_last_step_s():
    a, b = Solver(_case("odd")), Solver(_case("odd"))
    for n in (1, 3, 2):
        for _ in range(n):
            ra = a.step(1)
        assert ra == b.step(n)
    a.close()
    b.close()


def test_fp32_fluxes_keep_their_factors_apart():
    """S/V and |u.n| multiplied before the flux are rounded alike in every step, an
    error that adds up: 6.5e-9 rms of the limited cylinder flow's state after 10
    steps where the factors one by one leave 6.2e-9 (mean of 16 disturbed starts;
    its standard error is below 0.1e-9, and both forms round the same otherwise)."""
    err = []
    for seed in range(16):
        case = uc.cylinder2d(32, 16, nv=24, a=11.0, mach=5.0, kn=0.05, start="sheltered")
        n = len(case.W0)
        case.W0 = case.W0 * (1 + 0.02 * np.random.default_rng(seed).uniform(-1, 1, (n, 1)))
        a = Solver(case, limiter=1)
        b = Solver(case, limiter=1, precision=UGKS_FP32)
        a.step(10)
        b.step(10)
        W = a.W()
        mom = np.sqrt(2.0 * W[:, 0] * W[:, -1]).max()
        scale = np.array([W[:, 0].max(), mom, mom, W[:, -1].max()])
        err.append(np.sqrt((((b.W() - W) / scale) ** 2).mean()))
        a.close()
        b.close()
    print("FP32 form, rms error:", np.mean(err), flush=True)
    assert np.mean(err) <= 6.35e-9
