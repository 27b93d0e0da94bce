"""The small-channel direct conv's work-group shapes: 1, 2 and 4 output rows
(row counts around the thresholds, Ho not a multiple of them), each C_in and
C_out it serves, rows of whole dwords and odd ones, the patch in the weights'
place, strides 1 and above, bias, residual.  Sampled outputs against the
oracle, skip path equal to dense bit for bit, counts equal to the standalone
measurement's."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

# n, cin, h, w, cout, kh, kw, sh, sw, ph, pw
SHAPES = [
    (7, 3, 218, 64, 64, 7, 7, 2, 2, 3, 3),      # 763 rows: 2 per work-group, two blocks a row
    (7, 3, 219, 64, 64, 7, 7, 2, 2, 3, 3),      # 770 rows: 2, ragged
    (14, 3, 219, 50, 64, 7, 7, 2, 2, 3, 3),     # 1540 rows: 4, ragged, odd Wo
    (14, 3, 221, 51, 32, 3, 3, 2, 2, 1, 1),     # W C odd: element loads
    (16, 1, 100, 33, 16, 5, 5, 1, 1, 2, 2),     # one channel, C_out 16, stride 1, odd rows
    (16, 2, 97, 40, 32, 3, 4, 1, 3, 1, 0),      # even kernel width, stride 3
    (16, 4, 97, 40, 64, 3, 3, 1, 1, 1, 1),      # four channels
    (1, 1, 40, 501, 64, 8, 8, 2, 17, 0, 0),     # patch in the weights' place
    (2, 3, 9, 9, 64, 7, 7, 2, 2, 3, 3),         # most taps outside the image
    (3, 1, 5, 3, 16, 1, 1, 1, 1, 0, 0),         # tensor of 90 bytes
]


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_per_work_group(dt, shape):
    from paper_2511_19457_amd import abi
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dt]
    dev = torch.device("cuda")
    n, cin, h, wd, cout, kh, kw, sh, sw, ph, pw = shape
    d = abi.conv_desc(n, cin, h, wd, cout, kh, kw, sh, sw, ph, pw, dtype=tdt, has_bias=1)
    assert abi.sparoa_conv2d_tiling(d, 0) == (16, 32), "the direct kernel serves it"
    ho, wo = (h + 2 * ph - kh) // sh + 1, (wd + 2 * pw - kw) // sw + 1
    seed = 8000 + 10 * SHAPES.index(shape)
    x = synth.relu_normal((n, h, wd, cin), dt, seed)
    x[:, h // 2:] = 0
    w = synth.he_normal((cout, kh, kw, cin), kh * kw * cin, dt, seed + 1)
    b = synth.normal((cout,), dt, seed + 2)
    r = synth.normal((n, ho, wo, cout), dt, seed + 3)
    xd, wd_, bd, rd = x.to(dev), w.to(dev), b.to(dev), r.to(dev)
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(n * h * wd, cin, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(xd, n * h * wd, cin, 1, 8, 0, counts, mask)
    rows = n * ho * wo
    for res in (None, rd):
        yd = torch.full((n, ho, wo, cout), float("nan"), dtype=tdt, device=dev)
        ys, ym = torch.full_like(yd, float("nan")), torch.full_like(yd, float("nan"))
        abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, xd, wd_, bd, res, abi.ACT_RELU, None, yd)
        abi.sparoa_conv2d(d, abi.PATH_SKIP_MFMA, xd, wd_, bd, res, abi.ACT_RELU, mask, ys)
        nb = rows * (cout // 8)
        yc = torch.tensor([0, rows * cout, nb, nb], dtype=torch.int64, device=dev)
        commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
        abi.sparoa_conv2d_routed_measured(d, 2.0, 0.0, abi.ROUTE_BLOCK, counts, xd, wd_, bd, res,
                                          abi.ACT_RELU, mask, ym, yc, None, None, None, commit)
        want = torch.zeros(4, dtype=torch.int64, device=dev)
        wm = torch.zeros(abi.sparoa_mask_words(rows, cout, 1, 8), dtype=torch.int32, device=dev)
        abi.sparoa_measure_sparsity(yd, rows, cout, 1, 8, 0, want, wm)
        torch.cuda.synchronize()
        assert torch.equal(yd, ys) and torch.equal(yd, ym), shape
        assert torch.equal(yc, want) and not commit.any(), shape
        idx = np.unique(np.concatenate([
            np.random.default_rng(seed).integers(0, yd.numel(), size=3000), [0, yd.numel() - 1]]))
        yr, ar = oracle.conv2d_at(x, w, idx, n, cin, h, wd, cout, kh, kw, sh, sw, ph, pw, 1, 1, 1,
                                  bias=b, residual=None if res is None else r, act=1)
        got = yd.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
        assert np.all(np.abs(got - yr) <= RTOL[tdt] * ar + SUBNORMAL_STEP[tdt]), shape
