"""Launches of layers in 128 x 256 tiles whose rows may be split over two of
them, on the CPU: the library's launches are recorded instead of run
(launch_recorder.c), in a process of its own."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PROGRAM = r"""
import ctypes, json, sys
import torch                     # (its own libraries keep the real runtime)
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.recorded_name.restype = ctypes.c_char_p
from paper_2511_19457_amd import abi
out = []
for m, k, n, dt, path in json.loads(sys.argv[2]):
    d = abi.fc_desc(m, k, n, dt)
    need = abi.sparoa_fc_workspace_size(d, path)
    ws = torch.empty(max(16, need), dtype=torch.uint8)
    p, grid, got, err = 1 << 20, (ctypes.c_uint * 3)(), [], ""
    rec.forget_launches()
    try:
        abi.sparoa_fc(d, path, p, p, None, None, 0, p if path & 1 else None, p, ws)
    except abi.SparoaError as e:
        err = str(e)
    for i in range(rec.recorded_launches()):
        rec.recorded_grid(i, grid)
        got.append([rec.recorded_name(i).decode(), *grid])
    out.append([err, got])
print("LAUNCHES" + json.dumps(out))
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "launch_recorder.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-fPIC", "-shared", "-o", so,
                    os.path.join(HERE, "launch_recorder.c")], check=True)

    def run(calls):
        r = subprocess.run([sys.executable, "-c", PROGRAM, so, json.dumps(calls)],
                           cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout.split("LAUNCHES")[1])
    return run


# m, k, n of language-model output layers and generic wide FCs: one row of
# 128-row tiles and more than 256 column tiles, at remainders on both sides of
# half a round of 256, up to several rows of tiles
WIDE = [(1, 1024, 70000), (100, 1024, 81920), (128, 768, 81920), (128, 4096, 151936),
        (128, 4096, 163840), (7, 2048, 128256), (128, 768, 66000), (129, 1024, 81920),
        (256, 1024, 43520), (512, 1024, 22016), (300, 768, 50304), (384, 4096, 151936)]


@pytest.mark.parametrize("path", [0, 1])
@pytest.mark.parametrize("dt", [1, 2])
def test_no_launch_is_empty(launches, dt, path):
    calls = [[m, k, n, dt, path] for m, k, n in WIDE]
    for call, (err, got) in zip(calls, launches(calls)):
        assert not err and got, (call, err)
        assert all(x and y and z for _, x, y, z in got), (call, got)


# m, n and the 128 x 256 tiles of the first launch (0: one launch in all), by
# the tiles that whole rows of tiles within whole rounds leave over
SPLITS = [(33024, 256, 256), (3328, 3072, 252), (384, 22016, 172), (6528, 3072, 504),
          (65536 + 128 * 128, 256, 512), (65536, 256, 0), (32768 + 64 * 128, 256, 256), (32768 + 80 * 128, 256, 256),
          (32768 + 65 * 128, 256, 0), (32768 + 79 * 128, 256, 0), (512, 18944, 0),
          (1024, 11008, 0), (32768 + 129 * 128, 256, 0), (256, 43520, 0), (384, 50432, 0),
          (32768, 256, 0), (128, 81920, 0)]


def test_rows_split_by_the_tiles_left(launches):
    calls = [[m, 1024, n, 2, 0] for m, n, _ in SPLITS]
    for (m, n, head), (err, got) in zip(SPLITS, launches(calls)):
        assert not err, (m, n, err)
        grids = [x for name, x, _, _ in got if "igemm" in name]
        tiles = -(-m // 128) * -(-n // 256)
        if head:
            assert len(grids) == 2 and grids[0] == head and "2ELi4ELi4ELi4" in got[0][0], (m, n, got)
        else:
            assert grids == [tiles], (m, n, got)
