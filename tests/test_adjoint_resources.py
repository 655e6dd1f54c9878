"""Registers of the adjoint kernels of the FP32-shifted storage by rows, read from
the built library: three waves per SIMD (168 registers of 512) for the plain
kernel and the one with held planes, which two waves ran 5 to 8 % slower."""
import re

import pytest

from test_kernel_resources import kernel_resources


@pytest.mark.parametrize("model", ["D3Q95", "D2Q33", "D3Q19", "D3Q15"])
@pytest.mark.parametrize("hold", [0, 1])
def test_adjoint_by_rows_keeps_three_waves(model, hold):
    # k_adjoint<model, F32ST, FLAT = 0, NT = any, COLLIDE = 1, MARK = 0, HOLD>
    pat = re.compile(rf"k_adjointINS_\d+{model}E\w*F32STELb0ELb[01]ELb1ELb0ELb{hold}E")
    found = {n: v for n, v in kernel_resources().items() if pat.search(n)}
    assert len(found) == 2, sorted(found)
    for n, v in found.items():
        assert v["vgpr_count"] + v.get("agpr_count", 0) <= 168, (n, v)
        assert v["private_segment_fixed_size"] == 0, (n, v)
