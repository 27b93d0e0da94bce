"""Kernels of layers measured with and without count-commit words, on the CPU:
the launches are recorded instead of run (launch_recorder.c), in a process of
its own.  Without words a layer whose K the 64-row tiles do not split
takes those above 80, 128 and 192 few-tile work-groups (fewer than 3, fewer
than 9, more chunks), with words never."""
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
for m, k, n in json.loads(sys.argv[2]):
    for words in (0, 1):
        d = abi.conv_desc(1, k, 1, m, n, 1, 1, dtype=abi.BF16)
        ws = torch.empty(max(16, abi.sparoa_conv2d_workspace_size(d, 0)), dtype=torch.uint8)
        p, grid, got = 1 << 20, (ctypes.c_uint * 3)(), []
        rec.forget_launches()
        abi.sparoa_conv2d_routed_measured(d, 2.0, 0.0, 0, p, p, p, None, None, 0, p, p, p, None, ws,
                                          None, p if words else None)
        for i in range(rec.recorded_launches()):
            rec.recorded_grid(i, grid)
            got.append([rec.recorded_name(i).decode(), *grid])
        out.append(got)
print("LAUNCHES" + json.dumps(out))
"""

# m, k, n; work-groups without words (and whether in the few-tile kernel), with
LAYERS = [((320, 64, 64), 80, True, 80), ((321, 64, 64), 6, False, 84),
          ((3136, 128, 128), 98, False, 392), ((784, 128, 512), 104, False, 400),
          ((128, 512, 256), 128, True, 128), ((129, 512, 256), 12, False, 144),
          ((196, 1088, 128), 104, True, 104), ((3136, 640, 64), 49, False, 196),
          ((3136, 512, 64), 49, False, 196),
          ((196, 4608, 512), 208, True, 208)]


def test_kernels_by_commit_words(tmp_path):
    so = str(tmp_path / "launch_recorder.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-fPIC", "-shared", "-o", so,
                    os.path.join(HERE, "launch_recorder.c")], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, so, json.dumps([q[0] for q in LAYERS])],
                       cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    got = json.loads(r.stdout.split("LAUNCHES")[1])
    for (layer, direct, few, words), without, given in zip(LAYERS, got[::2], got[1::2]):
        assert [(x, "igemm_lk" in name) for name, x, _, _ in without] == [(direct, few)], (layer, without)
        assert [(x, "igemm_lk" in name) for name, x, _, _ in given] == [(words, True)], (layer, given)
