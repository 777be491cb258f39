"""Blocks of the measuring cast (f8_cast.hip), by the grids that reach the stand-in for the runtime's launch call of
test_launch_status.py: no GPU."""
import os
import subprocess
import sys

import pytest

from paper_2410_06511_amd import f8
from test_launch_status import stand_in  # noqa: F401 (a fixture)

CALL = r"""
import ctypes as C, sys
stand_in = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
l = C.CDLL(sys.argv[2])
rows, cols = map(int, sys.argv[3:])
x, scale, out, amax, ws = [C.c_void_p((k + 1) << 40) for k in range(5)]
l.f8_workspace_bytes.restype = C.c_size_t
stand_in.f8_test_reset(-1)
s = l.f8_cast_amax(x, C.c_int64(rows), C.c_int64(cols), C.c_int64(cols), scale, 0, out, C.c_int64(cols), None, C.c_int64(0), amax, ws,
                   C.c_size_t(l.f8_workspace_bytes(C.c_int64(rows), C.c_int64(cols))), None)
print(s, stand_in.f8_test_launches(), stand_in.f8_test_grid(0))
"""


@pytest.mark.parametrize("rows,cols,blocks", [
    (16, 16, 1), (256, 512, 16), (1024, 1600, 200), (1024, 4096, 512),     # a round of four chunks a thread
    (1024, 4608, 512), (1024, 6144, 512),                                  # and up to two chunks more
    (1024, 6160, 392), (1776, 3968, 434), (2176, 3248, 442),               # by the tiles: two rounds
    (2048, 4096, 512), (4096, 4096, 1024), (8192, 8192, 4096)])
def test_blocks_of_the_measuring_cast(stand_in, rows, cols, blocks):  # noqa: F811
    r = subprocess.run([sys.executable, "-c", CALL, stand_in, os.path.abspath(f8.LIB_PATH), str(rows), str(cols)], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr
    assert tuple(map(int, r.stdout.split())) == (0, 2, blocks)
