"""Temperature gradient with held planes where the grid is stored by rows: rows of
one wave, rows that end inside a wave, and rows whose last wave is mostly surplus
lanes.  Against the oracle's autograd: float64 within 1e-11 of the largest gradient
(the bar of the gradients in row groups), FP32-shifted within 1e-5 (that of the held
tubes).
"""
import numpy as np
import pytest
import torch

from oracle import lbm as olbm, velocity_sets as ovs
from synth_inputs import smooth_ic, smooth_noise, tube_ic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,extent,held", [
    ("D3Q95", (64, 6, 14), 5),
    ("D3Q95", (64, 5, 13), 5),
    ("D3Q95", (385, 2, 12), 5),
    ("D3Q95", (400, 2, 12), 5),
    ("D2Q33", (450, 20), 4),
    ("D3Q19", (128, 4, 8), 1),
])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("fp32s", 1e-5)])
def test_held_gradient_by_rows_matches_oracle_autograd(model, extent, held, precision, tol):
    from paper_1303_4624_amd import Simulation
    print("case", model, extent, precision, flush=True)
    D = len(extent)
    rho, U, th = tube_ic(extent, extent[-1] // 2, (2.0, 1.0), (1.0, 1.1))
    pr, pU, pth = smooth_ic(extent, seeds=(61, 62, 63, 64, 65)[:D + 2], amp_u=0.02, amp_rho=0.02,
                            amp_theta=0.02)
    rho, U, th = rho * pr, U + pU, th * pth
    v = ovs.velocity_set(model)
    lo = np.array([2.0] + [0.0] * D + [v.T0])
    hi = np.array([1.0] + [0.01] + [0.0] * (D - 1) + [1.1 * v.T0])
    target = 1.3 + 0.01 * smooth_noise(extent, 66)
    _, want, _ = olbm.loss_and_grad(v, rho, U, th * v.T0, 1.4, 5, target, (held, held, lo, hi))
    want = want.numpy()
    sim = Simulation(model, extent, 1.4, precision=precision)
    sim.set_fixed_planes(held, held, lo, hi)
    sim.init_fields(rho, U, th * sim.T0)
    ck = sim.run_checkpointed(5, 2, 1)
    g = 2.0 * (sim.moments()[0] - torch.as_tensor(target, device="cuda"))
    got, _ = sim.adjoint(5, 2, ck, rho, U, th * sim.T0, g, want_omega=False)
    sim.close()
    err = np.max(np.abs(got.cpu().numpy() - want)) / np.max(np.abs(want))
    print("dT error", err, flush=True)
    assert err <= tol
