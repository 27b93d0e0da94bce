"""FCs with more column tiles than the chip has compute units (language-model
output layers): one row of 128 x 256 tiles, full and ragged, and rows of tiles
whose remainder past whole rounds lies on both sides of the row split.  Sampled
outputs against the oracle, the skip path equal to the dense path bit for bit,
executed chunks counted on the CPU, and the fused output measurement equal to
the standalone one."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

# rows, columns (K = 768, the fewest chunks that take these tiles): one row of
# tiles with 257 and 320 columns of them; two rows of 170; three of 197
CASES = [(1, 256 * 256 + 1), (100, 81920), (128, 81920), (256, 43520), (300, 50304)]


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_wide_columns(dt, case):
    from paper_2511_19457_amd import abi
    tdt, dev = {"bf16": torch.bfloat16, "f16": torch.float16}[dt], torch.device("cuda")
    (m, n), k, seed = case, 768, 9300 + CASES.index(case)
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(m, k, generator=g).relu_().to(tdt)
    x[:, k // 2: k // 2 + 128] = 0    # chunks to skip everywhere
    x[m // 3:, : k // 4] = 0
    w = (torch.randn(n, k, generator=g) * k ** -0.5).to(tdt)
    b = synth.normal((n,), dt, seed + 1)
    xd, wd, bd = x.to(dev), w.to(dev), b.to(dev)
    d = abi.fc_desc(m, k, n, abi.BF16 if dt == "bf16" else abi.F16, has_bias=1)
    ws = torch.empty(max(16, abi.sparoa_fc_workspace_size(d, 0)), dtype=torch.uint8, device=dev)
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(m, k, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(xd, m, k, 1, 8, 0, counts, mask)
    y = torch.full((m, n), float("nan"), dtype=tdt, device=dev)
    ys = torch.full_like(y, float("nan"))
    done = torch.full((1,), -1, dtype=torch.int64, device=dev)
    abi.sparoa_fc(d, abi.PATH_DENSE_MFMA, xd, wd, bd, None, abi.ACT_RELU, None, y, ws)
    abi.sparoa_fc(d, abi.PATH_SKIP_MFMA, xd, wd, bd, None, abi.ACT_RELU, mask, ys, ws, done)
    torch.cuda.synchronize()
    what = f"{case} {dt}"
    assert torch.equal(y, ys), what
    rows = abi.sparoa_fc_tiling(d, abi.PATH_SKIP_MFMA)[0]
    u = (x != 0).reshape(m, k // 64, 64).any(2)
    assert int(done.item()) == sum(int(u[i:i + rows].any(0).sum()) for i in range(0, m, rows)), what
    idx = np.unique(np.concatenate([np.random.default_rng(seed).integers(0, m * n, size=600),
                                    [0, n - 1, m * n - 1], (m - 1) * n + np.arange(0, n, 997)]))
    yr, ar = oracle.conv2d_at(x.reshape(1, 1, m, k), w.reshape(n, 1, 1, k), idx, 1, k, 1, m, n,
                              1, 1, 1, 1, 0, 0, 1, 1, 1, bias=b, act=1)
    got = y.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
    assert np.all(np.abs(got - yr) <= RTOL[tdt] * ar + SUBNORMAL_STEP[tdt]), what
    if n % 64 == 0:
        nb, words = m * (n // 8), abi.sparoa_mask_words(m, n, 1, 8)
        want_c = torch.zeros(4, dtype=torch.int64, device=dev)
        want_m = torch.zeros(words, dtype=torch.int32, device=dev)
        abi.sparoa_measure_sparsity(y, m, n, 1, 8, 0, want_c, want_m)
        c = abi.conv_desc(1, k, 1, m, n, 1, 1, dtype=tdt, has_bias=1)
        ym = torch.full_like(y, float("nan"))
        yc = torch.tensor([0, m * n, nb, nb], dtype=torch.int64, device=dev)
        ymask = torch.full((words,), -1, dtype=torch.int32, device=dev)
        commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
        path = torch.zeros(1, dtype=torch.int32, device=dev)
        abi.sparoa_conv2d_routed_measured(c, 2.0, 0.0, abi.ROUTE_BLOCK, counts, xd, wd, bd, None,
                                          abi.ACT_RELU, mask, ym, yc, ymask, ws, path, commit)
        torch.cuda.synchronize()
        assert torch.equal(y, ym) and not commit.any(), what
        assert torch.equal(yc, want_c) and torch.equal(ymask, want_m), what
