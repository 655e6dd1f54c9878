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
        """cases: (model, extent, precision, streaming[, planes held at either end]);
        one dict of ints each."""
        lines = []
        for model, extent, precision, streaming, *hold in cases:
            ext = list(extent) + [1] * (3 - len(extent))
            lines.append(" ".join(str(x) for x in (
                len(extent), Q[model], *ext, {"fp64": 0, "fp32s": 1}[precision],
                {"ab": 0, "aa": 1}[streaming], *(hold or [0]))))
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


# Cells in flight a held CU needs at least: fewer leave HBM idle (D3Q95
# FP32-shifted 64x251x251 with one block of 64 cells 1308 us per step, unlimited 564).
ENOUGH = {("D3Q95", "fp32s", "ab"): 300, ("D3Q95", "fp32s", "aa"): 230,
          ("D3Q95", "fp64", "ab"): 150, ("D3Q95", "fp64", "aa"): 150,
          ("D3Q15", "fp32s", "ab"): 600, ("D3Q15", "fp32s", "aa"): 600}


def _enough(model, precision, streaming, nbytes):
    if (model, precision, streaming) == ("D3Q95", "fp32s", "aa") and nbytes < 1 << 30:
        return 300
    return ENOUGH.get((model, precision, streaming), 450 if precision == "fp32s" else 240)


@pytest.mark.parametrize("model,extents", [
    # odd row counts (rows do not pack), even ones, rows of one to many blocks, thin tubes
    ("D3Q95", [(64, 251, 251), (64, 250, 251), (128, 129, 129), (192, 129, 129), (256, 129, 129),
               (320, 111, 111), (400, 201, 201), (448, 161, 161), (11, 11, 20000), (5, 5, 60000),
               (3, 3, 90000), (16, 11, 20000), (130, 131, 129), (100, 1, 40000)]),
    ("D3Q19", [(64, 511, 511), (64, 512, 512), (128, 257, 257), (128, 256, 256), (192, 257, 257),
               (400, 161, 161), (448, 161, 161), (5, 5, 200000), (11, 11, 90000)]),
    ("D3Q15", [(64, 511, 511), (192, 257, 257), (384, 161, 161), (11, 11, 90000), (5, 7, 200000)]),
    ("D2Q33", [(64, 100001), (128, 40001), (128, 100000), (192, 50001), (400, 30001),
               (11, 500000), (2393, 3579)]),
])
@pytest.mark.parametrize("precision", ["fp64", "fp32s"])
@pytest.mark.parametrize("streaming", ["ab", "aa"])
def test_held_blocks_have_enough_cells(plans, model, extents, precision, streaming):
    cases = [(model, e, precision, streaming) for e in extents]
    held = 0
    for (_, e, _, _), p in zip(cases, plans(cases)):
        if p["resident"] == 0:
            continue
        held += 1
        cells = 1
        for n in e:
            cells *= n
        per_block = cells / p["blocks"]
        need = _enough(model, precision, streaming, p["bytes"])
        assert p["resident"] * per_block >= need, (e, p)
        assert p["resident"] <= 2 or (p["resident"] - 1) * per_block < need, (e, p)
    assert held > 0


def test_in_place_steps_of_d3q95_are_held_apart(plans):
    # the pushing step is held; the local one with it only where that was measured faster
    push_only = [((128, 128, 128), "fp64"), ((64, 250, 250), "fp64"), ((256, 256, 256), "fp64"),
                 ((192, 70, 60), "fp64"), ((400, 100, 100), "fp64"), ((200, 100, 100), "fp64"),
                 ((57, 176, 86), "fp32s"), ((350, 50, 40), "fp32s"), ((320, 80, 60), "fp32s"),
                 ((128, 128, 128), "fp32s")]
    both = [((17, 652, 269), "fp64"), ((192, 192, 192), "fp64"), ((320, 200, 200), "fp64"), ((384, 150, 150), "fp64"),
            ((256, 256, 256), "fp32s"), ((170, 145, 141), "fp32s")]
    for (e, prec), p in zip(push_only, plans([("D3Q95", e, pr, "aa") for e, pr in push_only])):
        assert p["resident"] > 0 and p["local"] == 0, (e, prec, p)
    for (e, prec), p in zip(both, plans([("D3Q95", e, pr, "aa") for e, pr in both])):
        assert p["resident"] > 0 and p["local"] == p["resident"], (e, prec, p)


# Narrow 2D grids: (extent, held) where several steps per launch were measured faster than
# single steps, and where they were slower, behind a full queue and from the host.
STRIPS = {
    "fp64": [((128, 4), 0), ((11, 800), 4), ((5, 1500), 0), ((16, 2400), 4), ((20, 800), 4),
             ((8, 2400), 4), ((600, 10), 0), ((3, 4000), 0), ((1, 500), 0)],
    "fp32s": [((128, 4), 0), ((11, 800), 4), ((5, 1500), 0), ((16, 2400), 4), ((20, 800), 4),
              ((25, 800), 4), ((36, 500), 4), ((300, 12), 0), ((600, 10), 0), ((3, 4000), 0)],
}
SINGLE = {
    "fp64": [((400, 16), 0), ((400, 16), 4), ((900, 20), 0), ((256, 20), 0), ((300, 12), 4),
             ((1000, 14), 4), ((40, 900), 0), ((60, 30), 0), ((64, 64), 0)],
    "fp32s": [((900, 20), 0), ((900, 16), 4), ((400, 16), 4), ((256, 20), 0), ((300, 12), 4),
              ((40, 900), 0), ((46, 42), 0), ((60, 30), 0), ((378, 24), 0), ((1423, 24), 0)],
}


@pytest.mark.parametrize("precision", ["fp64", "fp32s"])
def test_strips_are_taken_where_they_are_faster(plans, precision):
    got = plans([("D2Q33", e, precision, "ab", h) for e, h in STRIPS[precision]])
    for (e, h), p in zip(STRIPS[precision], got):
        assert p["strip_steps"] > 1 and 64 <= p["strip_threads"] <= 512, (e, h, p)
    got = plans([("D2Q33", e, precision, "ab", h) for e, h in SINGLE[precision]])
    for (e, h), p in zip(SINGLE[precision], got):
        assert p["strip_steps"] == 1, (e, h, p)
    assert all(p["strip_steps"] == 1 for p in plans(
        [("D2Q33", e, precision, "aa", h) for e, h in STRIPS[precision]]))


def test_wide_strips_of_the_gpu_test_are_planned(plans):
    from test_gpu_strips_wide import WIDE
    cases = [("D2Q33", e, p, "ab", h) for p, grids in WIDE.items() for e, h in grids]
    for case, p in zip(cases, plans(cases)):
        assert p["strip_steps"] > 1 and p["strip_threads"] > 256, (case, p)


@pytest.mark.parametrize("streaming", ["ab", "aa"])
def test_block_order_switches_on_the_grids_of_the_gpu_test(plans, streaming):
    from test_gpu_tune_blocks import ORDERED
    cases = [(m, e, p, streaming) for m, e, p, _, _ in ORDERED]
    for (m, e, _, flat, packed), p in zip(ORDERED, plans(cases)):
        assert p["order"] == 1, (m, e, p)
        assert (p["flat"] == 1) == flat and (p["rpb"] > 1) == packed, (m, e, p)


@pytest.mark.parametrize("model,extent,precision,most,limit", [
    # most: the block size the held steps of the set start from, limit: the largest
    ("D3Q95", (385, 71, 28), "fp32s", 256, 512), ("D3Q95", (400, 128, 128), "fp32s", 128, 512),
    ("D3Q19", (769, 120, 120), "fp32s", 256, 512), ("D2Q33", (804, 9000), "fp32s", 256, 512),
    ("D3Q95", (320, 80, 60), "fp32s", 256, 512), ("D3Q15", (1042, 100, 100), "fp32s", 256, 512),
])
def test_held_rows_take_the_blocks_with_the_fewest_idle_lanes(plans, model, extent, precision,
                                                              most, limit):
    p, = plans([(model, extent, precision, "aa")])
    nx = extent[0]

    def lanes(m):
        chunks = -(-nx // m)
        return chunks * (-(-(-(-nx // chunks)) // 64) * 64)
    fewest = min(lanes(m) for m in range(most, limit + 1, 64))
    assert p["resident"] > 0 and p["chunks"] * p["bx"] <= max(fewest, 1.1 * nx), p


def test_long_planes_are_stored_by_rows(plans):
    # states past 1 GB whose rows leave no slack for a partly empty last group: one group of the
    # whole plane up to 16384 cells, by rows past that; never more bytes than padded rows
    flat = [("D3Q95", (160, 50, 750), "fp64", "ab"), ("D3Q95", (32, 150, 1250), "fp32s", "ab"),
            ("D3Q19", (96, 50, 6250), "fp64", "aa"), ("D3Q95", (11, 11, 40000), "fp32s", "ab"),
            ("D3Q95", (31, 33, 9000), "fp32s", "aa"), ("D3Q95", (28, 30, 9000), "fp32s", "ab"),
            ("D3Q15", (30, 1219, 445), "fp64", "aa"), ("D2Q33", (20, 300001), "fp64", "aa")]
    rows = [("D2Q33", (96, 62501), "fp64", "ab"), ("D2Q33", (31, 200001), "fp64", "ab"),
            ("D2Q33", (224, 26786), "fp64", "aa"),
            ("D3Q95", (383, 250, 60), "fp64", "ab"), ("D3Q95", (224, 250, 100), "fp32s", "aa"),
            ("D3Q19", (160, 251, 600), "fp64", "ab"), ("D3Q95", (31, 33, 9000), "fp32s", "ab")]
    for cases, want in ((flat, 1), (rows, 0)):
        for (m, e, prec, st), p in zip(cases, plans(cases)):
            assert p["flat"] == want, (m, e, prec, st, p)
            align = 32 if e[0] >= 32 else 1
            padded = -(-e[0] // align) * align * Q[m] * (4 if prec == "fp32s" else 8)
            for n in e[1:]:
                padded *= n
            assert (1 << 30) < p["bytes"] <= padded, (m, e, prec, st, p)


def test_stores_of_the_smaller_sets_leave_the_cache_earlier(plans):
    # bytes of both buffers, measured faster with plain and with non-temporal stores
    plain = [("D2Q33", (1000, 1200), "fp32s"), ("D2Q33", (1000, 600), "fp64"),
             ("D3Q19", (128, 128, 66), "fp64"), ("D3Q95", (64, 64, 128), "fp32s"),
             ("D3Q95", (235, 64, 16), "fp64")]
    past = [("D2Q33", (1000, 1450), "fp32s"), ("D2Q33", (1024, 700), "fp64"),
            ("D3Q19", (128, 128, 156), "fp32s"), ("D3Q19", (128, 128, 76), "fp64"),
            ("D3Q95", (64, 64, 160), "fp32s")]
    assert [p["nt"] for p in plans([c + ("ab",) for c in plain])] == [0] * len(plain)
    assert [p["nt"] for p in plans([c + ("ab",) for c in past])] == [1] * len(past)
