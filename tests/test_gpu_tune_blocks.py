"""The alternative block order of the forward steps on the kinds of blocks the
grids of test_gpu_tune do not have: 2D rows and 2D flat groups, several rows
packed into a block, and several flat groups per block column in 3D.  That the
order is active on each (the grid holds a multiple of 8 slabs of blocks) is
checked from its launch plan without a GPU (test_launch_plans)."""
import pytest
import torch

from synth_inputs import smooth_ic

pytestmark = pytest.mark.gpu

# (model, extent, precision, flat groups, rows per block > 1)
ORDERED = [
    ("D2Q33", (128, 40), "fp32s", False, False),
    ("D2Q33", (1000, 64), "fp64", False, False),     # several blocks per row
    ("D2Q33", (100, 512), "fp32s", True, False),
    ("D3Q95", (128, 64, 40), "fp32s", False, True),
    ("D3Q19", (64, 96, 56), "fp64", False, True),
    ("D3Q95", (100, 70, 48), "fp32s", True, False),
]


@pytest.mark.parametrize("model,extent,precision,flat,packed", ORDERED)
@pytest.mark.parametrize("streaming", ["ab", "aa"])
def test_both_orders_give_the_same_bits(model, extent, precision, flat, packed, streaming):
    from paper_1303_4624_amd import Simulation
    print("case", model, extent, precision, streaming, flush=True)
    rho, U, th = smooth_ic(extent, seeds=tuple(range(81, 83 + len(extent))), amp_u=0.03)
    a, b = [Simulation(model, extent, 1.6, precision=precision, streaming=streaming)
            for _ in range(2)]
    for s in (a, b):
        s.init_fields(rho, U, th * s.T0)
    for order in (1, 0, 1):
        a.set_block_order(order)
        for _ in range(3):          # one by one: no strips
            a.step(1)
            b.step(1)
        assert torch.equal(a.get_populations(), b.get_populations()), order
    assert a.tune_step(13) in (0, 1)
    b.step(13)
    assert torch.equal(a.get_populations(), b.get_populations())
    a.close()
    b.close()
