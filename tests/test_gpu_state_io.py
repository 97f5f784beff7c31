"""Getting and setting the state: round trips in both forms, above and below the
size from which the GPU does the reordering, and the time they take against plain
copies of the same arrays."""

import time

import numpy as np
import pytest
import torch

import ugks_cases as uc
from paper_2606_15720_amd.ugks import UGKS_FP32, Batch, Solver, ugks_get_state

pytestmark = pytest.mark.gpu

STAGED = 2


def _tets(n, vel):
    case = uc.sod3d_tets(n=n, nv=4, jitter=0.15, seed=3)
    case.vel = vel
    return case


CASES = {
    "few values": lambda: uc.cavity2d(n=4, nv=7),
    "just few": lambda: uc.cavity2d(n=16, nv=8),          # 16,384 values
    "more": lambda: uc.cavity2d(n=17, nv=9),              # with pads
    "sparse": lambda: _tets(3, uc.locally_refined_grid(8, 4.0, 3, (1.2, 0.0, 0.0), 1.8)),
    "wide": lambda: uc.Case("hexes", uc.hex_box(4, grading=0.4, seed=1), uc.midpoint_grid(9, 4.0, 3),
                            uc.Gas(mu_ref=uc.hard_sphere_mu_ref(0.05)), [uc.BC(uc.BC_WALL) for _ in range(6)],
                            uc.uniform_W(64, 3, 1.0, (0.1, 0.0, 0.0), 1.0)),
    "pieces": lambda: _tets(6, uc.midpoint_grid(10, 4.0, 3)),  # 1.3e6 values: two pieces in the FP32 form
}


@pytest.mark.parametrize("flags", [0, STAGED])
@pytest.mark.parametrize("precision", [64, UGKS_FP32])
@pytest.mark.parametrize("which", CASES)
def test_state_round_trip(which, precision, flags):
    case = CASES[which]()
    rng = np.random.default_rng(1)
    shape = (case.mesh.n_cells, case.vel.nv)
    s = Solver(case, precision=precision, flags=flags)
    s.step(1)
    W0, h0, b0 = s.state()
    # what the library holds is what its moments are of
    w, u = case.vel.w, case.vel.u
    m = s.moments(1)
    np.testing.assert_allclose(h0 @ w, m[:, 0], rtol=1e-12)
    np.testing.assert_allclose((h0 * w) @ u, m[:, 1:1 + case.mesh.dim], rtol=0, atol=1e-12 * m[:, 0].max())
    h = rng.uniform(0.5, 1.5, shape)
    b = rng.uniform(0.5, 1.5, shape) if case.mesh.dim == 2 else np.zeros(shape)
    if precision == UGKS_FP32:
        h, b = h.astype(np.float32).astype(float), b.astype(np.float32).astype(float)
    s.set_state(W0, h, b)
    W1, h1, b1 = s.state()
    for x, y in ((W1, W0), (h1, h), (b1, b)):
        np.testing.assert_array_equal(x, y)
    # a restored state steps on as one that was never taken out
    r = Solver(case, precision=precision, flags=flags)
    r.step(1)
    s.set_state(W0, h0, b0)
    for _ in range(2):
        s.step(2)
        r.step(1)
        r.state()
        r.step(1)
    for x, y in zip(s.state(), r.state()):
        np.testing.assert_allclose(x, y, rtol=0, atol=1e-13 * np.abs(y).max() if precision == 64 else 1e-6 * np.abs(y).max())
    s.close()
    r.close()


def test_batch_state():
    cases = [uc.cavity2d(n=20, nv=10), uc.cavity2d(n=4, nv=7)]
    b, s = Batch(cases), Solver(cases[0])
    for n in (1, 2):
        b.step(n)
        s.step(n)
        for x, y in zip(b.state(0), s.state()):
            np.testing.assert_allclose(x, y, rtol=0, atol=1e-13 * np.abs(y).max())
    b.close()
    s.close()


def test_state_goes_at_the_rate_of_a_copy():
    # reordered by the CPU, value by value, h and b took 2 to 3 times as long as their copies
    s = Solver(uc.cavity2d(n=32, nv=28))
    state = s.state()
    host = [torch.from_numpy(x) for x in state[1:]]
    dev = [x.cuda() for x in host]

    def best(f):
        t = []
        for _ in range(15):
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)
    get, put = best(lambda: ugks_get_state(s.h, *state)), best(lambda: s.set_state(*state))
    down = best(lambda: [x.copy_(y) for x, y in zip(host, dev)])
    up = best(lambda: [y.copy_(x) for x, y in zip(host, dev)])
    print("get %.3f ms, its copies %.3f; set %.3f, copies %.3f" % tuple(1e3 * x for x in (get, down, put, up)),
          flush=True)
    assert get <= 1.6 * down and put <= 1.6 * up
    s.close()
