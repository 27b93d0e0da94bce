"""GEMM epilogues whose output rows start anywhere (C_out no multiple of 8):
every tile of the 64-channel-chunk kernel, its K splits and its partial
chunks, and the few-tile kernel's tiles in every dtype, with and without a
residual.  Sampled outputs (all of the last columns and rows among them)
against the oracle, the skip path equal to the dense path bit for bit, and
the bytes around y untouched."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

TDT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# m, k, n: 64 x 64 (whole chunks, partial ones, K split), 64 x 128 and its deep
# ring, 128 x 64, 128 x 128 twice, 128 x 256; then few-tile tiles up to 32 x 64
# (64 x 64 in fp32), one column past a tile and one short of it
WIDE = [(4000, 192, 253), (4000, 200, 130), (65, 2560, 5757), (6270, 192, 251),
        (3200, 2112, 509), (30721, 128, 61), (25000, 192, 127), (50100, 128, 127),
        (12500, 832, 510), (3000, 64, 1308)]
FEW = [(1, 64, 1), (17, 192, 17), (100, 1088, 127), (800, 128, 63), (1000, 640, 129),
       (2047, 128, 254), (2000, 320, 255)]


@pytest.mark.parametrize("res", [False, True])
@pytest.mark.parametrize("dt,shape", [(dt, s) for dt in ("bf16", "f16") for s in WIDE + FEW] +
                         [("f32", s) for s in FEW])
def test_ragged_columns(dt, shape, res):
    from paper_2511_19457_amd import abi
    tdt, dev = TDT[dt], torch.device("cuda")
    (m, k, n), seed = shape, 9500 + (WIDE + FEW).index(shape)
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(m, k, generator=g).relu_().to(tdt)
    x[m // 3: 2 * m // 3 + 1, : k // 2] = 0
    w = (torch.randn(n, k, generator=g) * k ** -0.5).to(tdt)
    b, r = synth.normal((n,), dt, seed + 1), synth.normal((m, n), dt, seed + 2)
    xd, wd, bd = x.to(dev), w.to(dev), b.to(dev)
    rd = r.to(dev) if res else None
    code = {"f32": abi.F32, "f16": abi.F16, "bf16": abi.BF16}[dt]
    d = abi.fc_desc(m, k, n, code, has_bias=1)
    ws = torch.empty(max(16, abi.sparoa_fc_workspace_size(d, 0)), dtype=torch.uint8, device=dev)
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(m, k, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(xd, m, k, 1, 8, 0, counts, mask)
    ys = []
    for path in (abi.PATH_DENSE_MFMA, abi.PATH_SKIP_MFMA):
        buf = torch.full((m * n + 128,), 7.0, dtype=tdt, device=dev)
        y = buf[64: 64 + m * n]
        abi.sparoa_fc(d, path, xd, wd, bd, rd, abi.ACT_RELU6, mask if path else None, y, ws)
        torch.cuda.synchronize()
        assert bool((buf[:64] == 7.0).all()) and bool((buf[64 + m * n:] == 7.0).all()), shape
        ys.append(y)
    assert torch.equal(*ys), (shape, dt)
    idx = np.unique(np.concatenate([np.random.default_rng(seed).integers(0, m * n, size=600),
                                    np.arange(min(m, 128)) * n + n - 1,
                                    (m - 1) * n + np.arange(n)[-130:]]))
    yr, ar = oracle.conv2d_at(x.reshape(1, 1, m, k), w.reshape(n, 1, 1, k), idx, 1, k, 1, m, n,
                              1, 1, 1, 1, 0, 0, 1, 1, 1, bias=b, residual=r if res else None, act=2)
    got = ys[0][torch.from_numpy(idx).to(dev)].double().cpu().numpy()
    assert np.all(np.abs(got - yr) <= RTOL[tdt] * ar + SUBNORMAL_STEP[tdt]), (shape, dt)
