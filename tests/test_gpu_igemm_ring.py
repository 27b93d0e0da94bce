"""The 64-channel-chunk GEMM's LDS ring: every tile the chooser takes, with
chunk counts around the ring's depth and a whole turn of it (1 chunk, fewer
than the stages, one more or less than a turn, several turns), ragged rows and
columns.  Sampled outputs against the oracle, the skip path equal to the dense
path bit for bit, and the fused output measurement equal to the standalone one
on the same bytes."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

# rows, columns: 64 x 64, 64 x 128 (deep ring from 32 chunks), 128 x 64,
# 128 x 128 (up to 256 tiles, more), 128 x 256; ragged rows, ragged columns
TILES = [(4000, 256), (6270, 256), (30721, 64), (25000, 128), (50100, 128), (12500, 512),
         (6270, 248), (30721, 72)]
CHUNKS = [1, 2, 3, 4, 5, 6, 7, 9, 10, 13]


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("tile", TILES)
def test_ring_depths(dt, tile):
    from paper_2511_19457_amd import abi
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dt]
    dev = torch.device("cuda")
    m, n = tile
    deep = tile[0] < 8000      # small enough for 33 chunks: the deep ring
    for chunks in ([1, 5, 31, 32, 33] if deep else CHUNKS[:6] if m > 20000 else CHUNKS):
        k = 64 * chunks
        seed = 7000 + 100 * TILES.index(tile) + chunks
        g = torch.Generator().manual_seed(seed)
        x = torch.randn(m, k, generator=g).relu_().to(tdt)
        x[m // 3: 2 * m // 3, : k // 2] = 0          # whole chunks to skip
        w = (torch.randn(n, k, generator=g) * k ** -0.5).to(tdt)
        b = synth.normal((n,), dt, seed + 1)
        xd, wd, bd = x.to(dev), w.to(dev), b.to(dev)
        d = abi.conv_desc(1, k, 1, m, n, 1, 1, dtype=tdt, has_bias=1)
        ws = torch.empty(max(16, abi.sparoa_conv2d_workspace_size(d, 0)), dtype=torch.uint8,
                         device=dev)
        counts = torch.zeros(4, dtype=torch.int64, device=dev)
        mask = torch.zeros(abi.sparoa_mask_words(m, k, 1, 8), dtype=torch.int32, device=dev)
        abi.sparoa_measure_sparsity(xd, m, k, 1, 8, 0, counts, mask)
        yd = torch.full((m, n), float("nan"), dtype=tdt, device=dev)
        ys = torch.full_like(yd, float("nan"))
        abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, xd, wd, bd, None, abi.ACT_RELU, None, yd, ws)
        abi.sparoa_conv2d(d, abi.PATH_SKIP_MFMA, xd, wd, bd, None, abi.ACT_RELU, mask, ys, ws)
        ym = torch.full_like(yd, float("nan"))
        nb = m * (n // 8)
        yc = torch.tensor([0, m * n, nb, nb], dtype=torch.int64, device=dev)
        words = abi.sparoa_mask_words(m, n, 1, 8)
        ymask = torch.full((words,), -1, dtype=torch.int32, device=dev)
        commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
        path = torch.zeros(1, dtype=torch.int32, device=dev)
        abi.sparoa_conv2d_routed_measured(d, 2.0, 0.0, abi.ROUTE_BLOCK, counts, xd, wd, bd, None,
                                          abi.ACT_RELU, mask, ym, yc, ymask, ws, path, commit)
        want_c = torch.zeros(4, dtype=torch.int64, device=dev)
        want_m = torch.zeros(words, dtype=torch.int32, device=dev)
        abi.sparoa_measure_sparsity(yd, m, n, 1, 8, 0, want_c, want_m)
        torch.cuda.synchronize()
        what = f"{tile} {dt} {chunks} chunks"
        assert torch.equal(yd, ys) and torch.equal(yd, ym), what
        assert torch.equal(yc, want_c) and torch.equal(ymask, want_m), what
        assert int(path.item()) == abi.PATH_DENSE_MFMA and not commit.any(), what
        idx = np.unique(np.concatenate([
            np.random.default_rng(seed).integers(0, m * n, size=800), [0, m * n - 1],
            (m - 1) * n + np.arange(min(n, 64))]))
        yr, ar = oracle.conv2d_at(x.reshape(1, 1, m, k), w.reshape(n, 1, 1, k), idx, 1, k, 1, m, n,
                                  1, 1, 1, 1, 0, 0, 1, 1, 1, bias=b, act=1)
        got = yd.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
        bound = RTOL[tdt] * ar + SUBNORMAL_STEP[tdt]
        assert np.all(np.abs(got - yr) <= bound), what
