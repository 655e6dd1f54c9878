"""Row groups and lane mapping of the update kernels, against the oracle, at the
edges of the choice: rows of one to many waves, one group per plane and several
with a partly empty last one, runs padded to whole lines and not, the first row
lengths stored by rows again, and every kernel that walks the groups (two-buffer,
in place, held planes, adjoint).

Bars: float64 1e-12 (the parity tests' bar).  In-place against two-buffer and
checkpointed against plain runs: bitwise."""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_run, oracle_run, rel_errors
from oracle import equilibrium as oeq, lbm as olbm, velocity_sets as ovs
from synth_inputs import grid_shape, smooth_ic

pytestmark = pytest.mark.gpu

EXTENTS = [
    ("D3Q95", (11, 11, 12)),      # one group per plane, its run padded to a line
    ("D3Q95", (6, 5, 7)),         # one group, run not padded (30 cells)
    ("D3Q95", (33, 32, 3)),       # one group of 1056 cells
    ("D3Q95", (100, 43, 2)),      # several groups, the last one partly empty
    ("D3Q95", (383, 5, 2)),       # the longest flat rows
    ("D3Q95", (385, 5, 2)),       # stored by rows, surplus lanes on the padding
    ("D3Q95", (128, 12, 3)),      # rows packed into blocks, groups of four rows
    ("D3Q95", (512, 4, 4)),       # 128 waves: the most whose work is split
    ("D3Q95", (192, 43, 1)),      # 129
    ("D2Q33", (11, 200)),         # 2D: groups of 128 rows
    ("D2Q33", (5, 3)),
    ("D2Q33", (383, 9)),
    ("D2Q33", (1000, 3)),         # by rows, two blocks per row
    ("D3Q15", (31, 70, 4)),
    ("D3Q19", (200, 7, 5)),
]


def new_sim(model, extent, omega, **kw):
    from paper_1303_4624_amd import Simulation
    return Simulation(model, extent, omega, **kw)


def _fields(extent):
    rng = np.random.default_rng(23)
    shape, D = grid_shape(extent), len(extent)
    return (1.0 + 0.05 * rng.standard_normal(shape), 0.03 * rng.standard_normal((D,) + shape),
            1.0 + 0.02 * rng.standard_normal(shape))


@pytest.mark.parametrize("model,extent", EXTENTS)
def test_update_matches_oracle_and_both_schemes_agree(model, extent):
    print("case", model, extent, flush=True)
    rho, U, th = _fields(extent)
    g = gpu_run(model, extent, 1.2, rho, U, th, 5)
    o = oracle_run(model, rho, U, th, 5, 1.2)
    errs = rel_errors(g, o, g[3])
    print("errors", errs, flush=True)
    assert max(errs) <= 1e-12
    for precision in ("fp64", "fp32s"):
        pops = []
        for streaming in ("ab", "aa"):
            sim = new_sim(model, extent, 1.2, precision=precision, streaming=streaming)
            sim.init_fields(rho, U, th * sim.T0)
            out = []
            for n in (1, 2):        # in place: both storage forms
                sim.step(n)
                out.append(sim.get_populations().cpu())
            sim.close()
            pops.append(out)
        assert all(torch.equal(a, b) for a, b in zip(*pops)), precision


@pytest.mark.parametrize("model,extent", [("D3Q95", (11, 11, 14)), ("D2Q33", (11, 150)),
                                          ("D2Q33", (7, 30)), ("D3Q95", (100, 20, 12))])
@pytest.mark.parametrize("streaming", ["ab", "aa"])
def test_held_planes_in_groups_match_oracle(model, extent, streaming):
    print("case", model, extent, streaming, flush=True)
    v = ovs.velocity_set(model)
    rho, U, th = smooth_ic(extent, amp_u=0.02)
    D = len(extent)
    lo = np.array([1.3] + [0.0] * D + [1.02 * v.T0])
    hi = np.array([0.9] + [0.0] * D + [0.97 * v.T0])
    sim = new_sim(model, extent, 1.3, streaming=streaming)
    sim.set_fixed_planes(4, 5, lo, hi)
    sim.init_fields(rho, U, th * sim.T0)
    sim.step(5)
    got = [x.cpu().numpy() for x in sim.moments()]
    sim.close()
    f = olbm.init_populations(v, rho, U, th * v.T0)
    want = [x.numpy() for x in oeq.moments(v, olbm.run(v, f, 1.3, 5, hold=(4, 5, lo, hi)))]
    errs = rel_errors(got, want, v.T0)
    print("errors", errs, flush=True)
    assert max(errs) <= 1e-12


@pytest.mark.parametrize("extent", [(11, 11, 6), (100, 20, 3), (36, 33, 2)])
def test_checkpoints_and_gradient_in_groups(extent):
    print("case", extent, flush=True)
    rho, U, th = smooth_ic(extent, amp_u=0.02)
    v = ovs.velocity_set("D3Q95")
    target = 1.0 + 0.01 * np.cos(np.arange(np.prod(extent))).reshape(rho.shape)
    _, gT, gw = olbm.loss_and_grad(v, rho, U, th * v.T0, 1.4, 5, target)
    sim = new_sim("D3Q95", extent, 1.4)
    sim.init_fields(rho, U, th * sim.T0)
    ck = sim.run_checkpointed(5, 2, 1)
    end = sim.get_populations()
    rho_n = sim.moments()[0]
    dT, dw = sim.adjoint(5, 2, ck, rho, U, th * sim.T0,
                         2.0 * (rho_n - torch.tensor(target, device="cuda")))
    eT = np.max(np.abs(dT.cpu().numpy() - gT.numpy())) / np.max(np.abs(gT.numpy()))
    print("errors", eT, abs(dw - gw) / abs(gw), flush=True)
    assert eT <= 1e-11 and abs(dw - gw) <= 1e-11 * abs(gw)
    sim.restore_checkpoint(5, 2, ck, 1)
    sim.step(3)
    assert torch.equal(sim.get_populations(), end)
    sim.close()
