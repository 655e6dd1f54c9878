"""The kernels that move populations in and out of the storage keep many loads in
flight: read from the instructions of the built library, the loads come in
batches before their stores, not one by one (which made them twice as slow on
grids of 20000 to 100000 cells)."""
import os
import re
import subprocess

import pytest

from test_kernel_resources import LIB, _device_objects, _section

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _copy_kernels(tmp_path):
    """{mangled name: loads and stores in order, as a string of L and S}"""
    out = {}
    for n, co in enumerate(_device_objects(_section(LIB, ".hip_fatbin"))):
        path = str(tmp_path / f"{n}.co")
        with open(path, "wb") as fh:
            fh.write(co)
        syms = subprocess.run([OBJDUMP, "--syms", path], capture_output=True, text=True,
                              check=True).stdout
        names = re.findall(r"(_ZN\S*k_(?:get_pop|set_pop|to_ab|from_ab)I\S*E)$", syms, re.M)
        names = sorted(x for x in set(names) if "D3Q95" in x and "F64T" in x)
        if not names:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + ",".join(names), path],
                              capture_output=True, text=True, check=True).stdout
        for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name = part[: part.index(">")]
            out[name] = "".join("L" if op == "load" else "S" for op in
                                re.findall(r"(?:global|flat|buffer)_(load|store)_", part))
    return out


def test_population_copies_load_in_batches(tmp_path):
    if not (os.path.exists(LIB) and os.path.exists(OBJDUMP)):
        pytest.skip("needs the built library and llvm-objdump")
    kernels = _copy_kernels(tmp_path)
    assert len(kernels) >= 6, sorted(kernels)
    for name, ops in kernels.items():
        assert ops.count("L") >= 95 and ops.count("S") >= 95, (name, len(ops))
        # a wave waits for memory about once per change from loads to stores
        assert ops.count("LS") <= 8, (name, ops)
