"""Device memory that the allocation-free cut holds: its one static array is
LODGS_NOALLOC_SCRATCH_BYTES (32 MiB) and 1 MiB (read from the array's symbol,
whose host-side stand-in has its size)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_static_array_of_the_allocation_free_cut():
    lib = os.path.join(ROOT, "paper_2507_01110_amd", "liblodgs.so")
    if not shutil.which("nm") or not os.path.exists(lib):
        pytest.skip("needs nm and the built library")
    src = open(os.path.join(ROOT, "include", "lodgs.h")).read()
    mib = int(re.search(r"#define LODGS_NOALLOC_SCRATCH_BYTES \((\d+)u << 20\)", src).group(1))
    rows = [l.split() for l in subprocess.check_output(["nm", "-S", lib], text=True).splitlines()]
    sizes = [int(r[1], 16) for r in rows if len(r) == 4 and r[2] in "bB" and "scratch" in r[3]]
    assert len(sizes) == 1 and mib << 20 <= sizes[0] <= (mib + 1) << 20, sizes
