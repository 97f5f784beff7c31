"""The blocked form of a batch (work items of a cell and a block of its velocities):
asked for by block_v, or found by the autotuner where the cells are few.  Bounds
are the single case's (1e-12 of the oracle, 1e-5 for the FP32 form)."""

import numpy as np
import pytest

import ugks_cases as uc
from oracle import Oracle
from paper_2606_15720_amd import ugks as U
from test_gpu_parity import _normwise

pytestmark = pytest.mark.gpu

EAGER = 8


def _tets(n, nv):
    case = uc.sod3d_tets(n=n, nv=nv, jitter=0.15, seed=3)
    left = case.mesh.cell_centroid[:, 0] < 0.5
    case.W0 = uc.uniform_W(case.mesh.n_cells, 3, np.where(left, 1.0, 0.6), (0.05, 0.0, 0.0),
                           np.where(left, 1.0, 0.9))
    return case


def _cases(dim):
    if dim == 3:
        return [_tets(1, 9), _tets(2, 6), _tets(1, 14)]
    return [uc.cavity2d(n=5, nv=16, kn=0.05), uc.channel2d(n=6, nv=9, kn=0.1), uc.cavity2d(n=3, nv=30, kn=0.05)]


@pytest.mark.parametrize("block_v", [64, 192, 640])  # half a wave of pairs, uneven blocks, one block for some cases
@pytest.mark.parametrize("dim", [2, 3])
def test_a_batch_in_blocks_follows_the_oracle(dim, block_v):
    cases = _cases(dim)
    for kw, tol in ((dict(), 1e-12), (dict(flags=EAGER, tile_cells=4), 1e-12), (dict(precision=U.UGKS_FP32), 1e-5)):
        b = U.Batch(cases, block_v=block_v, **kw)
        items = 0
        for i, c in enumerate(cases):
            bv = b.case_info(i)["block_v"]
            assert bv == block_v or c.vel.nv <= bv < block_v  # its whole set, with pads
            items += c.mesh.n_cells * -(-b.case_info(i)["nv_padded"] // bv)
        assert b.info["work_items"] >= items and b.info["tuned"] == 0
        for n in (1, 3):
            res = b.step(n)
        for i, c in enumerate(cases):
            o = Oracle(c)
            o.step(1)
            ro = o.step(3)
            err = _normwise(b.W(i), o.state(with_h=False)[0])
            print(dim, block_v, kw, c.name, err, flush=True)
            assert np.all(err <= tol)
            if tol < 1e-10:
                assert abs(res[i][1] - ro[1]) <= max(1e-12 * ro[1], 2.0 * tol)
        b.close()


def test_few_cells_with_many_velocities_are_tuned_to_blocks(tmp_path):
    # 6 cells x 28^3: one work-group per cell leaves 250 compute units idle
    U.ugks_autotune_clear()
    cases = [_tets(1, 28), _tets(1, 8)]
    a = U.Batch(cases)
    ia, bv = a.info, [a.case_info(i)["block_v"] for i in range(2)]
    print(ia, bv, flush=True)
    assert ia["tuned"] == 1 and ia["tune_timings"] > 0
    assert bv[0] <= 28 ** 3 // 2
    # the choice goes through a file, and gives the same schedule and results
    path = str(tmp_path / "tune.txt")
    U.ugks_autotune_save(path)
    U.ugks_autotune_clear()
    U.ugks_autotune_load(path)
    b = U.Batch(cases)
    ib = b.info
    assert ib["tune_timings"] == 0
    assert (ib["threads"], ib["work_items"], ib["grid"]) == (ia["threads"], ia["work_items"], ia["grid"])
    assert [b.case_info(i)["block_v"] for i in range(2)] == bv
    a.step(3)
    b.step(3)
    for i, c in enumerate(cases):
        np.testing.assert_array_equal(a.state(i)[1], b.state(i)[1])
        o = Oracle(c)
        o.step(3)
        assert np.all(_normwise(a.W(i), o.state(with_h=False)[0]) <= 1e-12)
    a.close()
    b.close()
    U.ugks_autotune_clear()


def test_a_case_that_fails_in_a_blocked_batch_keeps_its_step():
    bad = uc.cavity2d(n=8, nv=8, kn=0.05, lid=0.4)
    bad.gas.cfl = 4.0
    fine = uc.cavity2d(n=6, nv=8)
    s, good = U.Solver(bad), 0
    kept = s.W()
    for _ in range(100):
        try:
            s.step(1)
        except U.UGKSError:
            break
        kept, good = s.W(), good + 1
    s.close()
    assert good < 100
    c, d = U.Batch([fine, bad], block_v=64), U.Batch([fine], block_v=64)
    d.step(good + 2)
    with pytest.raises(U.UGKSError) as e:
        c.step(good + 2)
    assert e.value.code == U.UGKS_ENUMERIC
    np.testing.assert_array_equal(c.W(0), d.W(0))
    assert np.all(_normwise(c.W(1), kept) <= 1e-8)  # (rounding grows with the unstable mode)
    c.close()
    d.close()


def test_a_tuning_file_of_the_earlier_kernels_is_loaded_but_not_used(tmp_path):
    """Files from before the whole-cell step name their shapes without a mark; what
    they hold was timed on other kernels."""
    U.ugks_autotune_clear()
    case = uc.cavity2d(n=6, nv=8)
    lines = [f"case 2 64 {t} 36 64 : 32 16 {t}.5" for t in (64, 128, 256)] + ["batch 2 64 0 36 64 : 256"]
    path = tmp_path / "tune.txt"
    path.write_text("ugks-autotune 1\n" + "\n".join(lines) + "\n")
    U.ugks_autotune_load(str(path))
    b = U.Batch([case])
    assert b.info["tune_timings"] > 0
    b.close()
    out = tmp_path / "out.txt"
    U.ugks_autotune_save(str(out))
    assert set(lines) < set(out.read_text().splitlines())
    U.ugks_autotune_clear()
