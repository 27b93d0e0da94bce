"""The few-tile GEMM (small tiles whose waves split K): every tile of its rule
in every dtype it takes, with chunk counts around its wave counts and ring
depths, ragged rows and columns, partial channel chunks and padded, strided and
dilated taps.  Sampled outputs against the oracle, the skip path equal to the
dense path bit for bit, executed chunks counted on the CPU, and the fused
output measurement equal to the standalone one on the same bytes."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

TDT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# (n, c_in, h, w, c_out, k, stride, pad, dilation); chunks are 64 channels at
# 16 bits, 32 in fp32
SHAPES = [
    # 16 x 16 tiles: one pixel, one chunk; fewer chunks than waves; 16, 17 and
    # 18 chunks (4 waves, then 8); the longest of the rule at 16 bits
    (1, 64, 1, 1, 16, 1, 1, 0, 1), (1, 192, 1, 17, 24, 1, 1, 0, 1),
    (1, 1024, 1, 65, 64, 1, 1, 0, 1), (1, 1088, 1, 33, 72, 1, 1, 0, 1),
    (1, 128, 9, 7, 64, 3, 1, 1, 1), (1, 512, 3, 3, 64, 8, 1, 4, 1),
    # ragged columns that are no multiple of 8
    (2, 128, 6, 5, 19, 3, 1, 1, 1),
    # 16 x 32 and 16 x 64, short and long
    (1, 128, 28, 28, 128, 1, 1, 0, 1), (1, 128, 28, 28, 136, 3, 1, 1, 1),
    (1, 64, 56, 56, 64, 1, 1, 0, 1), (2, 64, 45, 39, 64, 3, 1, 1, 1),
    # 32 x 32 (under 4 chunks) and 32 x 64, stride and dilation
    (1, 128, 1, 2047, 256, 1, 1, 0, 1), (5, 128, 45, 39, 128, 3, 2, 1, 1),
    (2, 64, 60, 61, 64, 3, 1, 2, 2),
    # beyond them: 64 x 64 in fp32 (four waves), 528 tiles (the general kernel)
    (1, 320, 1, 4100, 192, 1, 1, 0, 1), (3, 64, 75, 75, 72, 3, 1, 1, 1),
    # partial chunks at 16 bits (C_in % 64 != 0)
    (1, 72, 14, 14, 40, 3, 1, 1, 1), (1, 48, 1, 300, 128, 1, 1, 0, 1),
]


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_few_tiles(dt, shape):
    from paper_2511_19457_amd import abi
    n, ci, h, w_, co, k, st, pd, dl = shape
    tdt, dev = TDT[dt], torch.device("cuda")
    seed = 9100 + SHAPES.index(shape)
    g = torch.Generator().manual_seed(seed)
    ho, wo = [(v + 2 * pd - dl * (k - 1) - 1) // st + 1 for v in (h, w_)]
    m = n * ho * wo
    x = torch.randn(n, h, w_, ci, generator=g).relu_()
    x[:, h // 2:, w_ // 3:, : ci // 2] = 0          # chunks to skip
    x = x.to(tdt)
    w = (torch.randn(co, k, k, ci, generator=g) * (ci * k * k) ** -0.5).to(tdt)
    b, r = synth.normal((co,), dt, seed + 1), synth.normal((m, co), dt, seed + 2)
    d = abi.conv_desc(n, ci, h, w_, co, k, k, st, st, pd, pd, dl, dl, dtype=tdt, has_bias=1)
    xd, wd, bd, rd = (t.to(dev) for t in (x, w, b, r))
    need = abi.sparoa_conv2d_workspace_size(d, 0)
    ws = torch.empty(max(16, need), dtype=torch.uint8, device=dev)
    pix = n * h * w_
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(pix, ci, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(xd, pix, ci, 1, 8, 0, counts, mask)
    y = torch.full((m, co), float("nan"), dtype=tdt, device=dev)
    ys = torch.full_like(y, float("nan"))
    done = torch.full((1,), -1, dtype=torch.int64, device=dev)
    abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, xd, wd, bd, rd, abi.ACT_RELU, None, y, ws)
    abi.sparoa_conv2d(d, abi.PATH_SKIP_MFMA, xd, wd, bd, rd, abi.ACT_RELU, mask, ys, ws, done)
    torch.cuda.synchronize()
    what = f"{shape} {dt}"
    assert torch.equal(y, ys), what

    # executed chunks: (row unit, chunk) pairs with some nonzero gathered input
    # (the fp32 chunk of a C_in that is no multiple of 32 crosses taps)
    c = 32 if dt == "f32" else 64
    if ci % c == 0 or dt != "f32":
        nz = (x.float() != 0).float().permute(0, 3, 1, 2)
        if ci % c:
            nz = torch.nn.functional.pad(nz, (0, 0, 0, 0, 0, c - ci % c))
        u = torch.nn.functional.unfold(nz, k, dilation=dl, padding=pd, stride=st)
        u = u.reshape(n, -1, c, k * k, ho * wo).amax(2).permute(0, 3, 1, 2).reshape(m, -1)
        rows = abi.sparoa_conv2d_tiling(d, abi.PATH_SKIP_MFMA)[0]
        want = sum(int(u[i:i + rows].amax(0).sum()) for i in range(0, m, rows))
        assert int(done.item()) == want, what

    idx = np.unique(np.concatenate([np.random.default_rng(seed).integers(0, m * co, size=600),
                                    [0, m * co - 1], (m - 1) * co + np.arange(min(co, 64))]))
    yr, ar = oracle.conv2d_at(x, w, idx, n, ci, h, w_, co, k, k, st, st, pd, pd, dl, dl, 1,
                              bias=b, residual=r, act=1)
    got = y.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
    assert np.all(np.abs(got - yr) <= RTOL[tdt] * ar + SUBNORMAL_STEP[tdt]), what

    if need:   # the workspace that the query names is still asked for
        with pytest.raises(Exception):
            abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, xd, wd, bd, rd, abi.ACT_RELU, None, y,
                              ws[: need - 16])
    if dt != "f32" and co % 64 == 0:
        nb = m * (co // 8)
        words = abi.sparoa_mask_words(m, co, 1, 8)
        want_c = torch.zeros(4, dtype=torch.int64, device=dev)
        want_m = torch.zeros(words, dtype=torch.int32, device=dev)
        abi.sparoa_measure_sparsity(y, m, co, 1, 8, 0, want_c, want_m)
        for fill in (0, -1):      # whatever the words held before
            ym = torch.full_like(y, float("nan"))
            yc = torch.tensor([0, m * co, nb, nb], dtype=torch.int64, device=dev)
            ymask = torch.full((words,), fill, dtype=torch.int32, device=dev)
            commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
            path = torch.zeros(1, dtype=torch.int32, device=dev)
            abi.sparoa_conv2d_routed_measured(d, 2.0 if fill else 0.0, 0.0, abi.ROUTE_BLOCK,
                                              counts, xd, wd, bd, rd, abi.ACT_RELU, mask, ym, yc,
                                              ymask, ws, path, commit)
            torch.cuda.synchronize()
            assert torch.equal(y, ym), what
            assert torch.equal(yc, want_c) and torch.equal(ymask, want_m), what
            assert not commit.any(), what
