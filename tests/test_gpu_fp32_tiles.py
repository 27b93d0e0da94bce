"""fp32 layers around the lines where the few-tile kernel's 64 x 64 tiles begin
and end: one chunk and two up to 256 tiles, 257 and 512 tiles, 513 to 768 and
769 to 1024 at the chunk count where these begin, more than 1024, and ragged
columns at 15 and 16 chunks.  A padded batch (three quarters of the samples
unused): sampled outputs against the oracle, the skip path equal to the dense
path bit for bit, executed chunks counted on the CPU."""
import numpy as np
import pytest
import torch

import oracle
import synth
from tests._util import RTOL, SUBNORMAL_STEP

pytestmark = pytest.mark.gpu

# samples, h, w, c_in, c_out, kernel
SHAPES = [(4, 25, 25, 32, 256, 1), (4, 25, 25, 64, 256, 1), (4, 16, 64, 64, 256, 1),
          (4, 25, 25, 480, 250, 1), (4, 25, 25, 512, 250, 1), (4, 57, 18, 32, 256, 3),
          (4, 64, 64, 64, 72, 1), (4, 64, 64, 32, 128, 1), (8, 32, 32, 64, 256, 1),
          (4, 47, 47, 352, 336, 1), (4, 47, 47, 384, 336, 1), (4, 47, 47, 384, 256, 1),
          (8, 47, 47, 736, 256, 1), (8, 47, 47, 768, 256, 1), (8, 48, 48, 96, 200, 3)]


@pytest.mark.parametrize("shape", SHAPES)
def test_fp32_tiles(shape):
    from paper_2511_19457_amd import abi
    n, h, w_, ci, co, k = shape
    dev, seed, m = torch.device("cuda"), 9900 + SHAPES.index(shape), n * h * w_
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, h, w_, ci, generator=g).relu_()
    x[n // 4:] = 0
    x[0, : h // 2, :, : ci // 2] = 0
    w = torch.randn(co, k, k, ci, generator=g) * (ci * k * k) ** -0.5
    b, r = synth.normal((co,), "f32", seed + 1), synth.normal((m, co), "f32", seed + 2)
    d = abi.conv_desc(n, ci, h, w_, co, k, k, 1, 1, k // 2, k // 2, dtype=torch.float32, has_bias=1)
    xd, wd, bd, rd = (t.to(dev) for t in (x, w, b, r))
    ws = torch.empty(max(16, abi.sparoa_conv2d_workspace_size(d, 0)), dtype=torch.uint8, device=dev)
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(m, ci, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(xd, m, ci, 1, 8, 0, counts, mask)
    y = torch.full((m, co), float("nan"), device=dev)
    ys = torch.full_like(y, float("nan"))
    done = torch.full((1,), -1, dtype=torch.int64, device=dev)
    abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, xd, wd, bd, rd, abi.ACT_RELU, None, y, ws)
    abi.sparoa_conv2d(d, abi.PATH_SKIP_MFMA, xd, wd, bd, rd, abi.ACT_RELU, mask, ys, ws, done)
    torch.cuda.synchronize()
    assert torch.equal(y, ys), shape
    u = torch.nn.functional.unfold((x != 0).float().permute(0, 3, 1, 2), k, padding=k // 2)
    u = u.reshape(n, ci // 32, 32, k * k, h * w_).amax(2).permute(0, 3, 1, 2).reshape(m, -1)
    rows = abi.sparoa_conv2d_tiling(d, abi.PATH_SKIP_MFMA)[0]
    assert int(done.item()) == sum(int(u[i:i + rows].amax(0).sum()) for i in range(0, m, rows)), shape
    idx = np.unique(np.concatenate([
        np.random.default_rng(seed).integers(0, m * co // 4, size=500),
        np.random.default_rng(seed + 1).integers(m * co // 4, m * co, size=200),
        (m - 1) * co + np.arange(min(co, 64))]))
    yr, ar = oracle.conv2d_at(x, w, idx, n, ci, h, w_, co, k, k, 1, 1, k // 2, k // 2, 1, 1, 1,
                              bias=b, residual=r, act=1)
    got = y.reshape(-1)[torch.from_numpy(idx).to(dev)].double().cpu().numpy()
    assert np.all(np.abs(got - yr) <= RTOL[torch.float32] * ar + SUBNORMAL_STEP[torch.float32]), shape
