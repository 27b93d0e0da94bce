"""Layers measured without count-commit words (every work-group adds to the
counters itself) on both sides of the rule that takes them out of the few-tile
GEMM: work-groups around its limits, with and without a K split, partial channel
chunks, ragged rows, C_out % 64 == 0 and not.  Counts and bitmap equal a
standalone measurement of the output, dense and skip routes agree bit for bit,
and the output agrees with the oracle and with the call that gives words."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

# m, k, n; work-groups of the few-tile kernel
SHAPES = [(320, 64, 64),       # 80
          (321, 64, 64),       # 84
          (81, 128, 256), (128, 512, 256),      # 96; 128
          (129, 512, 256), (196, 1152, 128),    # 144; 104
          (3136, 128, 128), (784, 72, 512),     # 392; 400 of 32 x 32
          (3135, 264, 128),    # 196 of 32 x 64
          (196, 4608, 512),    # 208, K split over work-groups in 64-row tiles
          (100, 2560, 136)]    # the same, C_out % 64 != 0


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_direct_commits(dt, shape):
    from paper_2511_19457_amd import abi
    tdt, dev = {"f16": torch.float16, "bf16": torch.bfloat16}[dt], torch.device("cuda")
    (m, k, n), seed = shape, 9900 + SHAPES.index(shape)
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(m, k, generator=g).relu_()
    x[m // 2:, : k // 2] = 0
    w = torch.randn(n, k, generator=g) * k ** -0.5
    w[n // 2: n // 2 + 8] = 0                # zero blocks of y, and scattered zeros
    x, w = x.to(tdt), w.to(tdt)
    b = synth.normal((n,), dt, seed + 1)
    b[n // 2: n // 2 + 8] = 0
    r = synth.normal((m, n), dt, seed + 2)
    r[:, n // 2: n // 2 + 8] = 0
    xd, wd, bd, rd = (t.to(dev) for t in (x, w, b, r))
    d = abi.conv_desc(1, k, 1, m, n, 1, 1, dtype=tdt, has_bias=1)
    ws = torch.empty(max(16, abi.sparoa_conv2d_workspace_size(d, 0)), dtype=torch.uint8, device=dev)
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(m, k, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(xd, m, k, 1, 8, 0, counts, mask)
    nb, words = m * (n // 8), abi.sparoa_mask_words(m, n, 1, 8)
    idx = np.unique(np.concatenate([np.random.default_rng(seed).integers(0, m * n, size=600),
                                    [0, m * n - 1], (m - 1) * n + np.arange(min(n, 64))]))
    yr, ar = oracle.conv2d_at(x.reshape(1, 1, m, k), w.reshape(n, 1, 1, k), idx, 1, k, 1, m, n,
                              1, 1, 1, 1, 0, 0, 1, 1, 1, bias=b, residual=r, act=1)
    # (two sums of K products in fp32, rounded once each to 16 bits)
    tol = RTOL[tdt] * ar + SUBNORMAL_STEP[tdt]
    seen = []
    for thr in (2.0, 0.0):      # routed dense, routed to skip
        for bitmap in (True, False):
            for words_given in (False, True):
                y = torch.full((m, n), float("nan"), dtype=tdt, device=dev)
                yc = torch.tensor([0, m * n, nb, nb], dtype=torch.int64, device=dev)
                ymask = torch.full((words,), -1, dtype=torch.int32, device=dev)
                commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
                path = torch.zeros(1, dtype=torch.int32, device=dev)
                abi.sparoa_conv2d_routed_measured(
                    d, thr, 0.0, abi.ROUTE_BLOCK, counts, xd, wd, bd, rd, abi.ACT_RELU, mask, y, yc,
                    ymask if bitmap else None, ws, path, commit if words_given else None)
                want_c = torch.zeros(4, dtype=torch.int64, device=dev)
                want_m = torch.zeros(words, dtype=torch.int32, device=dev)
                abi.sparoa_measure_sparsity(y, m, n, 1, 8, 0, want_c, want_m)
                torch.cuda.synchronize()
                what = (shape, dt, thr, bitmap, words_given)
                assert torch.equal(yc, want_c) and int(path.item()) == (thr == 0.0), what
                if bitmap:
                    assert torch.equal(ymask, want_m), what
                got = y.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
                assert np.all(np.abs(got - yr) <= tol), what
                seen.append((words_given, y))
    for words_given in (False, True):
        same = [y for q, y in seen if q == words_given]
        assert all(torch.equal(same[0], y) for y in same), (shape, dt, words_given)
