"""The autotuner of a batch times every lane count, not the smallest alone."""

import pytest

import ugks_cases as uc
from paper_2606_15720_amd import ugks as U

pytestmark = pytest.mark.gpu


def test_large_velocity_sets_take_more_than_one_wave_per_cell():
    # 8 x 1,296 tets x 20^3, FP64: 1.75 ms per step with 64 lanes, 1.3 with 256
    U.ugks_autotune_clear()
    b = U.Batch([uc.sod3d_tets(n=6, nv=20) for _ in range(8)])
    print(b.info, flush=True)
    assert b.info["tuned"] == 1 and b.info["threads"] > 64
    b.step(1)
    b.close()
    U.ugks_autotune_clear()
