"""Several steps per launch on narrow 2D grids whose strips take more than 256
threads (two waves per SIMD, the upper half of the strip's LDS), along x and y,
more than 16 cells across, with a partly empty last strip and held planes: n
steps in one call against n calls of one step, bitwise.  That each grid takes
such strips is checked from its launch plan without a GPU (test_launch_plans)."""
import numpy as np
import pytest
import torch

from synth_inputs import grid_shape

pytestmark = pytest.mark.gpu

# (extent, planes held at either end) by storage type
WIDE = {
    "fp64": [((16, 2403), 4), ((20, 803), 4), ((11, 801), 0), ((8, 2405), 0), ((20, 20), 0),
             ((301, 12), 0), ((8193, 8), 0)],
    "fp32s": [((16, 2403), 0), ((20, 803), 0), ((25, 805), 4), ((36, 501), 4), ((36, 67), 0),
              ((19, 23), 4), ((301, 12), 0), ((603, 10), 0)],
}


@pytest.mark.parametrize("precision,extent,hold",
                         [(p, e, h) for p, cases in WIDE.items() for e, h in cases])
def test_n_steps_equal_single_steps_in_wide_strips(precision, extent, hold):
    from paper_1303_4624_amd import Simulation
    print("case", precision, extent, hold, flush=True)
    rng = np.random.default_rng(37)
    shape = grid_shape(extent)
    rho = 1.0 + 0.05 * rng.standard_normal(shape)
    U = 0.03 * rng.standard_normal((2,) + shape)
    th = 1.0 + 0.02 * rng.standard_normal(shape)
    sims = [Simulation("D2Q33", extent, 1.2, precision=precision) for _ in range(2)]
    for sim in sims:
        if hold:
            sim.set_fixed_planes(hold, hold, [1.1, 0.0, 0.0, 1.02 * sim.T0],
                                 [0.95, 0.0, 0.0, 0.98 * sim.T0])
        sim.init_fields(rho, U, th * sim.T0)
    one, many = sims
    for n in (3, 5, 14):
        for _ in range(n):
            one.step(1)
        many.step(n)
        assert torch.equal(one.get_populations(), many.get_populations()), n
    for sim in sims:
        sim.close()
