"""Vector registers of the element-parallel kernels whose lanes walk their rows alone, one float or 16-bit
elements each (fewer lanes a row than rows loaded ahead): what they hold decides how many waves a SIMD keeps in
flight (512 registers, given out in steps of 8), and these kernels live on that. 100,000,000 rows of one float
took 449 us at 69 registers and 353 at 50. (fp32 rows of 2 to 8 floats gain more from padded batches than they
lose by the registers, and are not held to a number here.)"""
import re
import subprocess

import pytest

from paper_2404_03019_amd import build

# (reduction, mode, vec, lanes, storage, ids): waves per SIMD
KERNELS = {
    ("RED_SUM", "SRC_ROWS", 1, 1, "ELEM_F32", "int64_t"): 9,
    ("RED_MAX", "SRC_ROWS", 1, 1, "ELEM_F32", "int64_t"): 9,
    ("RED_SUM", "SRC_ROWS", 1, 4, "ELEM_F32", "int64_t"): 7,
    ("RED_SUM", "SRC_ROWS", 8, 1, "ELEM_BF16", "int32_t"): 5,
    ("RED_SUM", "SRC_ROWS", 8, 4, "ELEM_BF16", "int32_t"): 4,
    ("RED_SUM", "SRC_ROWS", 4, 1, "ELEM_BF16", "int32_t"): 9,
    ("RED_SUM", "SRC_ROWS", 4, 2, "ELEM_F16", "int32_t"): 7,
    ("RED_MAX", "SRC_ROWS", 4, 2, "ELEM_BF16", "int64_t"): 7,
}


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    d = tmp_path_factory.mktemp("registers")
    lines = ['#include "common.h"', '#include "ep_kernel.h"', "namespace geot { namespace {"]
    for red, mode, vec, lanes, elem, ids in KERNELS:
        lines.append(f"template __global__ void ep_kernel<{red}, {mode}, {vec}, 1, {lanes}, {elem}, {ids}, false>(const EpArgs);")
    (d / "k.hip").write_text("\n".join(lines + ["} }", ""]))
    flags = [f for f in build.FLAGS if not f.startswith("-W")]
    subprocess.run([build.HIPCC, *flags, "-I", build.CSRC, "--cuda-device-only", "-S", str(d / "k.hip"), "-o", str(d / "k.s")],
                   check=True, capture_output=True, timeout=300)
    text = (d / "k.s").read_text()
    found = re.findall(r"\.name:\s+\S+ep_kernel\S+.*?\.vgpr_count:\s+(\d+)\s+\.vgpr_spill_count:\s+(\d+)", text, re.S)
    assert len(found) == len(KERNELS)
    return dict(zip(KERNELS, [(int(a), int(b)) for a, b in found]))


@pytest.mark.parametrize("kernel", list(KERNELS), ids=lambda k: "-".join(map(str, k)))
def test_waves_in_flight(registers, kernel):
    used, spilled = registers[kernel]
    assert spilled == 0 and 512 // ((used + 7) // 8 * 8) >= KERNELS[kernel], f"{used} registers"
