"""One launch or two for the attention's backward (f8_attn.hip), by the grids that reach the stand-in for the runtime's launch
call of test_launch_status.py: no GPU, 256 compute units."""
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
B, S, Hq, Hkv = map(int, sys.argv[3:])
p = [C.c_void_p((k + 1) << 40) for k in range(11)]
i64, wq, wk = C.c_int64, C.c_int64(Hq * 128), C.c_int64(Hkv * 128)
stand_in.f8_test_reset(-1)
s = l.f8_sdpa_bwd_rows(p[0], wq, p[1], wk, p[2], wk, p[3], wq, p[4], wq, p[5], i64(B), i64(S), i64(Hq), i64(Hkv), i64(128), p[6], wq, p[7], wk,
                       p[8], wk, p[9], None, p[10], C.c_size_t(1 << 40), None)
print(s, *[stand_in.f8_test_grid(k) for k in range(2)])
"""


@pytest.mark.parametrize("B,S,Hq,Hkv,one", [
    # a tile to a sequence and head: in one launch while all blocks find a unit, or long enough for a second round
    (16, 16, 8, 8, True), (17, 16, 8, 8, False), (30, 48, 8, 8, False), (17, 104, 8, 8, False), (17, 112, 8, 8, True), (31, 256, 8, 8, True),
    (16, 16, 8, 2, True), (17, 56, 8, 2, False), (17, 64, 8, 2, True), (27, 56, 8, 2, False), (28, 40, 8, 2, False), (28, 48, 8, 2, True), (31, 256, 8, 2, True), (32, 256, 8, 8, False),
    # several: by the blocks to a unit
    (4, 1000, 16, 16, True), (21, 512, 8, 8, True), (22, 512, 8, 8, False), (1, 8192, 8, 8, True), (1, 8192, 32, 8, False)])
def test_one_launch_or_two(stand_in, B, S, Hq, Hkv, one):  # noqa: F811
    r = subprocess.run([sys.executable, "-c", CALL, stand_in, os.path.abspath(f8.LIB_PATH), *map(str, (B, S, Hq, Hkv))], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr
    blocks = (S + 255) // 256 * Hq * B
    # delta's kernel takes 128 rows a block
    assert tuple(map(int, r.stdout.split())) == ((0, (B * S * Hq + 127) // 128, 2 * blocks) if one else (0, blocks, blocks))
