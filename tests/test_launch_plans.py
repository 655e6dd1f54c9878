"""Launch plans: what the host code chooses for a grid, printed by a small program
built around lbm_api.cpp with the kernel launchers stubbed out (no GPU needed)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1303_4624_amd", "csrc")
ROCM = "/opt/rocm"
Q = {"D2Q33": 33, "D3Q95": 95, "D3Q19": 19, "D3Q15": 15}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "lib", "libamdhip64.so")):
        pytest.skip("needs g++ and the HIP runtime library")
    exe = str(tmp_path_factory.mktemp("plans") / "print_plans")
    srcs = [os.path.join(CSRC, "lbm_model_host.cpp"),
            os.path.join(ROOT, "tests", "host_plans", "print_plans.cpp"),
            os.path.join(ROOT, "tests", "sanitize", "launcher_stubs.cpp")]
    cmd = [gxx, "-std=c++20", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, *srcs, "-L", os.path.join(ROCM, "lib"),
           f"-Wl,-rpath,{ROCM}/lib", "-lamdhip64", "-lquadmath", "-o", exe]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                         timeout=600)
    assert res.returncode == 0, res.stdout[-4000:]

    def ask(cases):
        """cases: (model, extent, precision, streaming); one dict of ints each."""
        lines = []
        for model, extent, precision, streaming in cases:
            ext = list(extent) + [1] * (3 - len(extent))
            lines.append(" ".join(str(x) for x in (
                len(extent), Q[model], *ext, {"fp64": 0, "fp32s": 1}[precision],
                {"ab": 0, "aa": 1}[streaming])))
        run = subprocess.run([exe], input="\n".join(lines) + "\n", stdout=subprocess.PIPE,
                             text=True, timeout=300)
        assert run.returncode == 0
        out = [dict((k, int(v)) for k, v in (f.split("=") for f in line.split()))
               for line in run.stdout.splitlines()]
        assert len(out) == len(lines)
        return out
    return ask


# Grids past the cache whose plans hold 1 to 8 blocks per CU.
HELD = [
    ("D3Q95", (384, 384, 384), "fp32s", "ab"), ("D3Q95", (256, 256, 256), "fp32s", "aa"),
    ("D3Q95", (256, 256, 256), "fp64", "ab"), ("D3Q95", (192, 192, 192), "fp64", "aa"),
    ("D3Q19", (256, 256, 256), "fp32s", "ab"), ("D3Q19", (192, 257, 257), "fp32s", "ab"),
    ("D3Q19", (128, 257, 257), "fp64", "ab"), ("D3Q19", (64, 511, 511), "fp32s", "ab"),
    ("D2Q33", (8192, 8192), "fp64", "ab"), ("D2Q33", (128, 40001), "fp64", "aa"),
]


@pytest.mark.parametrize("unit", [512, 1280])
def test_reserved_lds_holds_the_planned_number_of_blocks(plans, unit):
    # a CU has 160 KB, given out in units
    got = set()
    for case, p in zip(HELD, plans(HELD)):
        assert p["resident"] > 0 and p["lds"] > 0, case
        block = -(-p["lds"] // unit) * unit
        assert 160 * 1024 // block == p["resident"], (case, p)
        got.add(p["resident"])
    assert len(got) >= 4, got
