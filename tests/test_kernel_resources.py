"""Registers and scratch memory of the kernels beside the aggregation kernel (CPU only: hipcc cross-compiles for
gfx950), from the compiler's own report.  A spilled register is a trip to memory inside the loops that these kernels
are; what is spilled today, and why that is borne, is written out below."""
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2204_02662_amd" / "csrc"
FILES = ("epp_rows", "epp_combine", "epp_combine_split", "epp_prepare", "epp_prepare_small", "epp_partition", "epp_tiles")


@pytest.fixture(scope="module")
def usage(tmp_path_factory):
    """{file: {mangled name: (scratch bytes per lane, wavefronts per SIMD)}}"""
    d = tmp_path_factory.mktemp("resources")

    def one(f):
        out = subprocess.run(
            ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
             "-packed-fp32-ops", f"-I{ROOT / 'include'}", f"-I{CSRC}", "-c", str(CSRC / (f + ".hip")), "-o", f"{f}.o",
             "-Rpass-analysis=kernel-resource-usage"], cwd=d, capture_output=True, text=True, timeout=900)
        assert out.returncode == 0, out.stderr[-3000:]
        found, name, scratch = {}, None, 0
        for line in out.stderr.splitlines():
            if m := re.search(r"Function Name: (\S+)", line):
                name = m.group(1)
            elif m := re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line):
                scratch = int(m.group(1))
            elif m := re.search(r"Occupancy \[waves/SIMD\]: (\d+)", line):
                found[name] = (scratch, int(m.group(1)))
        return f, found

    with ThreadPoolExecutor(4) as pool:
        return dict(pool.map(one, FILES))


def test_scratch_memory(usage):
    for f, kernels in usage.items():
        assert kernels, f
        for name, (scratch, _) in kernels.items():
            limit = 0
            if "k_weight_gradient_rowsILi4ELi4E" in name:
                limit = 84   # 128 x 128: the product's 256 accumulators and eight pairs of rows ahead leave no room
            elif "k_prepare_smallILb0E" in name:
                limit = 132  # one workgroup, launched once per graph
            assert scratch <= limit, (f, name, scratch)


def test_wavefronts_of_the_row_kernel(usage):
    rows = {n: o for n, (_, o) in usage["epp_rows"].items() if "k_aggregate_rows" in n}
    assert len(rows) == 20  # ten shapes of a source row, with and without an inner path
    assert min(rows.values()) >= 8, rows


def test_input_gradient_workgroups_at_once(usage):
    """The launch starts as many workgroups as the chip holds at once, by this table (epp_combine.hip: resident)."""
    at_once = {(2, 1): 4, (2, 2): 4, (2, 4): 3, (4, 1): 4, (4, 2): 4, (4, 4): 3, (6, 1): 4, (6, 2): 4, (6, 4): 3, (8, 1): 3,
               (8, 2): 3, (8, 4): 2, (12, 1): 3, (12, 2): 2, (12, 4): 2, (16, 1): 2, (16, 2): 2, (16, 4): 2}
    found = {}
    for name, (_, waves) in usage["epp_combine"].items():
        if m := re.search(r"k_input_gradient_rowsILi(\d+)ELi(\d)E", name):
            found[int(m.group(1)), int(m.group(2))] = waves
    assert set(found) == set(at_once)
    for shape, n in at_once.items():
        assert found[shape] >= n, (shape, found[shape])
