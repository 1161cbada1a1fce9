"""The tile limit of the symmetric work lists bounds every array that is sized by it.

SDBIE_SYM_MAX_TILES sets it at compile time.  The staging kernels hold one
count per 64 tiles in LDS, kSymMaxTiles / 256 rows per thread of the scan, and
T^2 ranks in the source records' memory: a limit that these can follow compiles,
one past the records' memory does not, and neither can reach a device.
"""
import os
import re
import subprocess

import pytest

from paper_2110_10749_amd import build


def check(limit):
    cmd = [build.hipcc(), *build.FLAGS, f"-DSDBIE_SYM_MAX_TILES={limit}", "-fsyntax-only", "--cuda-device-only",
           os.path.join(build.CSRC, "stage.hip")]
    return subprocess.run(cmd, capture_output=True, text=True, timeout=110)


@pytest.mark.parametrize("limit,ok", [(2048, True), (8192, True), (16384, False), (2049, False)])
def test_arrays_follow_the_tile_limit_or_do_not_compile(limit, ok):
    r = check(limit)
    assert (r.returncode == 0) == ok, r.stderr[-2000:]
    assert ok or "static assertion failed" in r.stderr or "static_assert" in r.stderr


def test_no_array_is_sized_by_a_number_of_its_own():
    with open(os.path.join(build.CSRC, "stage.hip")) as f:
        text = f.read()
    assert not re.search(r"\b(2048|524288) */ *(64|256)", text)
    # the host refuses too many tiles before the first kernel that writes rows of them
    assert text.index("P.ntiles > kSymMaxTiles") < text.index("(k_mask_rows,")
