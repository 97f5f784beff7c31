"""Cells of five to eight faces on a symmetric tensor velocity set, against
the oracle: padded faces of mixed meshes, odd and sparse sets, far-field ghost
rows, the limiter, local steps, b, and the face fluxes after a call of several
steps.  Bounds are the parity tests' (1e-12 on the state, 1e-13 on the face
fluxes): the same sums in another order."""

import numpy as np
import pytest

import ugks_cases as uc
from oracle import Oracle
from paper_2606_15720_amd.ugks import UGKS_FP32, Solver, ugks_profile_enable, ugks_profile_read
from test_gpu_parity import LOCAL_DT, STAGED, TRACK, _compare_step, _normwise, _normwise_F

pytestmark = pytest.mark.gpu


def _merged(mesh, groups):
    """The mesh with each group of cells made one cell."""
    label = np.arange(mesh.n_cells)
    for g in groups:
        label[list(g)] = min(g)
    keep, label = np.unique(label, return_inverse=True)
    m = mesh.contiguous()
    vol = np.bincount(label, m.cell_volume)
    cen = np.stack([np.bincount(label, m.cell_volume * m.cell_centroid[:, d]) / vol
                    for d in range(m.dim)], axis=1)
    fc = np.where(m.face_cells >= 0, label[m.face_cells], m.face_cells)
    inner = fc[:, 0] != fc[:, 1]
    return uc.Mesh(m.dim, vol, cen, fc[inner], m.face_area[inner], m.face_normal[inner],
                   m.face_centroid[inner], m.face_shift[inner], m.face_bc[inner],
                   m.face_bc_id[inner]).contiguous()


def _hexes(nv, far=(), n=(4, 3, 3), vel=None, K=0):
    mesh = uc.hex_box(*n, grading=0.5, seed=5)
    bcs = [uc.BC(uc.BC_WALL, 1.0, (0.0, 0.0 if s in (2, 3) else 0.05 * s, 0.0), 1.0 + 0.1 * s) for s in range(6)]
    for s in far:
        mesh.face_bc[mesh.face_bc_id == s] = uc.BC_FARFIELD
        bcs[s] = uc.BC(uc.BC_FARFIELD, 0.8, (0.2, 0.0, 0.1), 1.2)
    case = uc.Case("hexes", mesh, vel or uc.midpoint_grid(nv, 4.0, 3),
                   uc.Gas(mu_ref=uc.hard_sphere_mu_ref(0.05)), bcs, None, 0)
    case.gas.K = K
    case.W0 = uc.uniform_W(mesh.n_cells, 3, 1.0, (0.1, 0.0, 0.0), 1.0, **({"K": K} if K else {}))
    case.W0 *= 1.0 + 0.1 * np.random.default_rng(3).uniform(-1, 1, (mesh.n_cells, 1))
    return case


def _case(which):
    if which == "walls":
        return _hexes(7), 0, dict(limiter=1, limiter_k=0.5)
    if which == "far_field":  # 12^3 / 2 pairs: more than the largest work-group
        return _hexes(12, far=(0, 3)), 0, {}
    if which == "local_steps":
        return _hexes(8, far=(1,)), LOCAL_DT, {}
    if which == "sparse":
        return _hexes(0, vel=uc.locally_refined_grid(6, 4.0, 3, (0.9, 0.0, -0.3), 1.2)), 0, {}
    if which == "internal":
        return _hexes(8, K=2), 0, {}
    case = uc.channel2d(n=6, nv=9, kn=0.05, u_in=0.6)
    x = case.mesh.cell_centroid
    def near(*pts):
        return [int(np.argmin(((x - x.mean(0) - p) ** 2).sum(1))) for p in pts]
    lo, hi = x.min(0), x.max(0)
    hx, hy = (np.unique(np.round(x[:, d], 9))[1] - lo[d] for d in (0, 1))
    c = lo - x.mean(0)
    block = near(c, c + (hx, 0), c + (0, hy), c + (hx, hy))       # eight faces, in a corner
    c = hi - x.mean(0)
    row = near(c, c - (hx, 0))                                    # six faces
    case.mesh = _merged(case.mesh, [block, row])
    case.W0 = uc.uniform_W(case.mesh.n_cells, 2, 1.0, (0.1, 0.0), 1.0)
    return case, 0, {}


@pytest.mark.parametrize("which", ["walls", "far_field", "local_steps", "sparse", "internal", "merged_quads"])
def test_wide_cells_follow_the_oracle(which):
    case, flags, lim = _case(which)
    most = np.bincount(case.mesh.face_cells[case.mesh.face_cells >= 0]).max()
    assert most == (8 if which == "merged_quads" else 6)
    _compare_step(case, 4, flags=flags, **lim)
    case, flags, lim = _case(which)
    o = Oracle(case, local_dt=bool(flags & LOCAL_DT), **lim)
    s = Solver(case, flags=flags, **lim)
    assert s.info["fused"] == 0
    o.step(3)
    s.step(3)
    err = _normwise_F(s.faces()[0], o.faces()[0])
    print(which, "face fluxes", err, flush=True)
    assert np.all(err <= 1e-13), err
    s.close()


def test_wide_cells_fp32_tracking_and_graphs_against_the_staged_sweep():
    # FP32 storage with FP64 arithmetic on both: they part by roundings of f
    case = _hexes(8, far=(2,))
    a, b = Solver(case, precision=UGKS_FP32), Solver(case, precision=UGKS_FP32, flags=STAGED)
    a.step(4)
    b.step(4)
    assert np.all(_normwise(a.W(), b.W()) <= 1e-6)
    a.close()
    b.close()
    a, b = Solver(case, flags=TRACK | 32), Solver(case, flags=STAGED | TRACK)
    for _ in range(3):
        a.step(2)
        b.step(2)
    fa, fb = a.boundary_flux(), b.boundary_flux()
    assert fa[1] == fb[1]
    assert np.all(np.abs(np.asarray(fa[0]) - np.asarray(fb[0])) <= 1e-12 * np.abs(np.asarray(fb[0])).max())
    assert np.all(_normwise(a.W(), b.W()) <= 1e-12)
    a.close()
    b.close()


@pytest.mark.parametrize("which", ["far_field", "merged_quads"])
def test_wide_cells_fp32_form_takes_ghost_states_in_fp64(which):
    """The first step of the FP32 form starts from f that both sweeps hold alike and
    computes in FP64, so the states part by FP64 roundings; ghost values rounded to
    FP32 (6e-8 each) showed at some 1e-10 of W."""
    case = _case(which)[0]
    a, b = Solver(case, precision=UGKS_FP32), Solver(case, precision=UGKS_FP32, flags=STAGED)
    a.step(1)
    b.step(1)
    err = _normwise(a.W(), b.W())
    fa, fb = a.faces()[0], b.faces()[0]
    print(which, err, _normwise_F(fa, fb), flush=True)
    assert np.all(err <= 1e-14)
    assert np.all(_normwise_F(fa, fb) <= 1e-13)
    a.close()
    b.close()


def test_few_cells_take_every_xcd():
    """27 cells x 40^3 and 216 x 20^3 have the same gradients to compute and write.  On
    one XCD of eight the few cells' took over three times as long; both fill the
    GPU, so they should differ by no more than a half."""
    def gradients(n, nv):
        s = Solver(_hexes(nv, n=(n, n, n)), flags=STAGED)
        s.step(3)
        best = np.inf
        for _ in range(5):
            ugks_profile_enable(s.h, True)
            s.step(4)
            n_launch, ms = ugks_profile_read(s.h)["micro_gradient"]
            best = min(best, ms / n_launch)
        s.close()
        return best
    few, many = gradients(3, 40), gradients(6, 20)
    print("gradients of 27 x 40^3 and 216 x 20^3, ms:", few, many, flush=True)
    assert few <= 1.5 * many


@pytest.mark.parametrize("nv,lim", [(4, {}), (7, dict(limiter=1, limiter_k=0.5))])  # 1 and 3 waves of pairs
def test_many_wide_cells_with_few_velocities(nv, lim):
    # enough cells that lanes come from the pairs alone: more of them than pairs
    _compare_step(_hexes(nv, far=(2,), n=(17, 16, 16)), 2, **lim)
