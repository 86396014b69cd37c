"""The d = 128 forward's walks without a decode state spill no vector register.

Their state tiles fill the register file (236 and 252 of 256 registers): with
the loads and stores of a decode state in the same kernels both spilled, which
cost every call 2-4 us.  The counts come from the metadata of the code objects
in libhla.so (built here from this repository's sources).  CPU only.
"""
import os
import re
import subprocess

import pytest

from tests.test_store_data_hazard import LIB, _gfx950_code_objects

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _spilled(tmp_path):
    """{kernel: spilled vector registers} of the library."""
    got = {}
    for i, blob in enumerate(_gfx950_code_objects(LIB)):
        path = tmp_path / f"co{i}.o"
        path.write_bytes(blob)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            symbol = re.search(r"\.symbol:\s*(\S+)\.kd", kernel).group(1)
            got[symbol] = int(re.search(r"\.vgpr_spill_count:\s*(\d+)", kernel).group(1))
    return got


@pytest.mark.skipif(not os.path.exists(LIB), reason="libhla.so is not built")
@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
def test_stateless_walks_do_not_spill(tmp_path):
    walks = {s: n for s, n in _spilled(tmp_path).items() if re.search(r"k_walk_ws_(first|out)(?!ILb1E)", s)}
    assert len(walks) == 2, sorted(walks)
    assert not any(walks.values()), walks
