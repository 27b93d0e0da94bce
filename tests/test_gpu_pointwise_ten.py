"""Pointwise layers of 9 and 10 channel blocks (129 to 160 channels) in the
kernel's ten-block instance, for each count of k-steps it has and for the one
it leaves to twelve: dense against the oracle, skip equal to dense bit for bit,
with and without a residual, the fused measurement equal to the standalone."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("cin", [24, 40, 120, 136])          # 1, 2, 4 and 8 k-steps
@pytest.mark.parametrize("cout", [136, 144, 152, 160])
def test_ten_blocks(dt, cin, cout):
    from paper_2511_19457_amd import abi
    tdt, dev = {"bf16": torch.bfloat16, "f16": torch.float16}[dt], torch.device("cuda")
    # (from 48 channels the kernel takes 32768 pixels or more)
    h, seed = (182, 41) if cin >= 48 else (33, 40)
    m = h * h
    g = torch.Generator().manual_seed(seed + cin + cout)
    x = torch.randn(m, cin, generator=g).relu_()
    x[m // 3: m // 2] = 0
    x = x.to(tdt)
    w = (torch.randn(cout, cin, generator=g) * cin ** -0.5).to(tdt)
    b, r = synth.normal((cout,), dt, seed), synth.normal((m, cout), dt, seed + 1)
    d = abi.conv_desc(1, cin, h, h, cout, 1, 1, dtype=tdt, has_bias=1)
    assert abi.sparoa_conv2d_tiling(d, abi.PATH_DENSE_BW) == (16, 32)
    xd, wd, bd, rd = (t.to(dev) for t in (x, w, b, r))
    idx = np.unique(np.concatenate([
        np.random.default_rng(seed).integers(0, m * cout, size=500), [0, m * cout - 1],
        (m - 1) * cout + np.arange(cout)]))
    for res_h, res_d in ((None, None), (r, rd)):
        y = torch.full((m, cout), float("nan"), dtype=tdt, device=dev)
        ys = torch.full_like(y, float("nan"))
        abi.sparoa_conv2d(d, abi.PATH_DENSE_BW, xd, wd, bd, res_d, abi.ACT_RELU6, None, y)
        abi.sparoa_conv2d(d, abi.PATH_SKIP_BW, xd, wd, bd, res_d, abi.ACT_RELU6, None, ys)
        torch.cuda.synchronize()
        assert torch.equal(y, ys)
        yr, ar = oracle.conv2d_at(x, w.reshape(cout, 1, 1, cin), idx, 1, cin, h, h, cout, 1, 1,
                                  bias=b, residual=res_h, act=2)
        got = y.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
        assert np.all(np.abs(got - yr) <= RTOL[tdt] * ar + SUBNORMAL_STEP[tdt])
        nb, words = m * (cout // 8), abi.sparoa_mask_words(m, cout, 1, 8)
        want_c = torch.zeros(4, dtype=torch.int64, device=dev)
        want_m = torch.zeros(words, dtype=torch.int32, device=dev)
        abi.sparoa_measure_sparsity(y, m, cout, 1, 8, 0, want_c, want_m)
        counts = torch.tensor([0, m * cin, m, m], dtype=torch.int64, device=dev)
        yc = torch.tensor([0, m * cout, nb, nb], dtype=torch.int64, device=dev)
        ymask = torch.full((words,), -1, dtype=torch.int32, device=dev)
        commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
        path = torch.zeros(1, dtype=torch.int32, device=dev)
        ym = torch.full_like(y, float("nan"))
        abi.sparoa_conv2d_routed_measured(d, 2.0, 1e9, abi.ROUTE_BLOCK, counts, xd, wd, bd, res_d,
                                          abi.ACT_RELU6, None, ym, yc, ymask, None, path, commit)
        torch.cuda.synchronize()
        assert torch.equal(y, ym) and torch.equal(yc, want_c) and torch.equal(ymask, want_m)
        assert not commit.any()
