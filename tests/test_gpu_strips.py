"""Several steps per launch of narrow 2D grids: n steps in one call against n
calls of one step (bitwise) and the oracle (float64, 1e-12), on strips along x
and y, one strip holding the whole grid, a partly empty last strip, axes shorter
than a displacement and held planes; step counts that leave remainders; and
captured calls, whose replays need the state in the buffer single steps leave
it in."""
import numpy as np
import pytest
import torch

from gpu_helpers import rel_errors
from oracle import equilibrium as oeq, lbm as olbm, velocity_sets as ovs
from synth_inputs import grid_shape

pytestmark = pytest.mark.gpu

STATES = ([1.1, 0.0, 0.0, 1.02], [0.95, 0.0, 0.0, 0.98])   # (rho, U, theta)


def _sim(extent, precision, hold, **kw):
    from paper_1303_4624_amd import Simulation
    rng = np.random.default_rng(31)
    shape = grid_shape(extent)
    rho = 1.0 + 0.05 * rng.standard_normal(shape)
    U = 0.03 * rng.standard_normal((2,) + shape)
    th = 1.0 + 0.02 * rng.standard_normal(shape)
    sim = Simulation("D2Q33", extent, 1.2, precision=precision, **kw)
    held = [s[:3] + [s[3] * sim.T0] for s in STATES]
    if hold:
        sim.set_fixed_planes(hold, hold, *held)
    sim.init_fields(rho, U, th * sim.T0)
    return sim, (rho, U, th), held


@pytest.mark.parametrize("extent,hold", [
    ((128, 4), 0), ((4, 131), 0), ((300, 12), 0), ((16, 90), 0),
    ((30, 3), 0), ((5, 7), 0), ((1, 50), 0), ((3, 2), 0),
    ((11, 200), 4), ((60, 9), 4), ((7, 21), 4),
])
@pytest.mark.parametrize("precision", ["fp64", "fp32s"])
def test_n_steps_equal_single_steps(extent, hold, precision):
    print("case", extent, hold, precision, flush=True)
    one, _, _ = _sim(extent, precision, hold)
    many, (rho, U, th), held = _sim(extent, precision, hold)
    total = 0
    for n in (3, 4, 16, 23):
        for _ in range(n):
            one.step(1)
        many.step(n)
        total += n
        assert torch.equal(one.get_populations(), many.get_populations()), n
    if precision == "fp64":
        v = ovs.velocity_set("D2Q33")
        f = olbm.init_populations(v, rho, U, th * v.T0)
        f = olbm.run(v, f, 1.2, total, hold=(hold, hold, *held) if hold else None)
        want = [x.numpy() for x in oeq.moments(v, f)]
        errs = rel_errors([x.cpu().numpy() for x in many.moments()], want, v.T0)
        print("errors", errs, flush=True)
        assert max(errs) <= 1e-12
    one.close()
    many.close()


@pytest.mark.parametrize("n", [6, 10])
def test_captured_steps_replay(n):
    print("case", n, flush=True)
    stream = torch.cuda.Stream()
    eager, _, _ = _sim((128, 4), "fp64", 0)
    sim, _, _ = _sim((128, 4), "fp64", 0, stream=stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sim.step(n)
    for _ in range(3):
        graph.replay()
        eager.step(n)
        torch.cuda.synchronize()
        assert torch.equal(sim.get_populations(), eager.get_populations())
    eager.close()
    sim.close()
