"""The kernels that fill a state from fields or populations and copy it hand each
XCD a contiguous range of blocks: every cell is written once whatever the number
of blocks (fewer than 8, a multiple of 8 and not, a partly filled last one), so
populations and moments come back as they went in, in both storage types and
schemes, also after an odd number of in-place steps."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,extent", [
    ("D3Q95", (5, 3, 2)), ("D3Q95", (64, 8, 4)), ("D3Q95", (31, 29, 11)), ("D3Q95", (128, 16, 9)),
    ("D2Q33", (257, 8)), ("D2Q33", (96, 85)), ("D3Q19", (40, 13, 11)),
])
@pytest.mark.parametrize("precision,tol", [("fp64", 0.0), ("fp32s", 1.2e-7)])
@pytest.mark.parametrize("streaming", ["ab", "aa"])
def test_populations_return_as_they_went_in(model, extent, precision, tol, streaming):
    from paper_1303_4624_amd import Simulation
    print("case", model, extent, precision, streaming, flush=True)
    shape, D = tuple(reversed(extent)), len(extent)
    g = torch.Generator(device="cuda").manual_seed(5)
    noise = lambda s: torch.rand(s, dtype=torch.float64, device="cuda", generator=g) - 0.5  # noqa: E731
    rho, U, th = 1.0 + 0.02 * noise(shape), 0.02 * noise((D,) + shape), 1.0 + 0.02 * noise(shape)
    sim = Simulation(model, extent, 1.4, precision=precision, streaming=streaming)
    sim.init_fields(rho, U, th * sim.T0)
    r, u, t = sim.moments()
    # the fields come back to the rounding of Q stored values (float32: of the deviations)
    bar = 1e-13 if precision == "fp64" else 2e-6
    assert (r - rho).abs().max() <= bar and (u - U).abs().max() <= bar
    assert (t - th * sim.T0).abs().max() <= bar
    for n in (0, 1):
        sim.step(n)
        f = sim.get_populations()
        assert bool(torch.isfinite(f).all())
        sim.set_populations(f)
        back = sim.get_populations()
        # float32 storage of f - w rho0: half a unit in the last place of |f| <= 1
        assert (back - f).abs().max() <= tol
    sim.close()
