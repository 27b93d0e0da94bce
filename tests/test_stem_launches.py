"""Work-groups of the small-channel direct conv, on the CPU: its launches are
recorded instead of run (launch_recorder.c), in a process of its own."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

PROGRAM = r"""
import ctypes, json, sys
import torch                     # (its own libraries keep the real runtime)
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.recorded_name.restype = ctypes.c_char_p
from paper_2511_19457_amd import abi
out = []
for n, ci, h, w, co, k, s in json.loads(sys.argv[2]):
    d = abi.conv_desc(n, ci, h, w, co, k, k, s, s, k // 2, k // 2, dtype=abi.BF16)
    p, grid, got = 1 << 20, (ctypes.c_uint * 3)(), []
    rec.forget_launches()
    abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, p, p, None, None, 0, None, p)
    for i in range(rec.recorded_launches()):
        rec.recorded_grid(i, grid)
        got.append([rec.recorded_name(i).decode(), *grid])
    out.append(got)
print("LAUNCHES" + json.dumps(out))
"""

# n, c_in, h, w, c_out, kernel, stride, and the work-groups: one, two or three
# 16-pixel blocks a row at more rows than CUs (4 or 2 rows a work-group, so
# that no wave is without a block), the same at fewer, then four and more
# blocks a row
STEMS = [(119, 4, 12, 12, 64, 7, 2, 238), (300, 4, 12, 12, 64, 7, 2, 600),
         (43, 1, 28, 28, 64, 7, 2, 172), (18, 4, 28, 28, 64, 7, 2, 252), (20, 2, 40, 40, 16, 5, 2, 200),
         (12, 2, 40, 40, 16, 5, 2, 240), (15, 2, 40, 40, 64, 7, 1, 300),
         (1, 3, 80, 80, 64, 3, 2, 40), (4, 2, 96, 96, 64, 3, 2, 192), (1, 3, 224, 224, 64, 7, 2, 112),
         (8, 3, 224, 224, 64, 7, 2, 448), (32, 3, 224, 224, 64, 7, 2, 896)]


def test_no_wave_without_a_block(tmp_path):
    so = str(tmp_path / "launch_recorder.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-fPIC", "-shared", "-o", so,
                    os.path.join(HERE, "launch_recorder.c")], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, so, json.dumps([s[:-1] for s in STEMS])],
                       cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    for stem, got in zip(STEMS, json.loads(r.stdout.split("LAUNCHES")[1])):
        grids = [x for name, x, _, _ in got if "conv_small_c" in name]
        assert grids == [stem[-1]], (stem, got)
