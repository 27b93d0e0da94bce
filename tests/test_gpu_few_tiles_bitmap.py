"""The few-tile GEMM's output bitmap: bits set and cleared by atomics (tiles
narrower than 64 channels, C_out that is no multiple of 64) or stored as
bytes, in every tile that a measured layer takes: rows that share words, long
rows, grids around the direct commits, partial channel chunks, few and many
chunks.  The output equals the unmeasured call's bit for bit, counts and
bitmap equal a standalone measurement of it, whatever the bitmap's words held
before, on both routes."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

# m, k, n.  n % 64 == 0: one and several rows of tiles under 256 channels, 16
# and 64 of each width, 33 to 64 tiles, 256 to 512 channels, 1024 up, 32 rows.
# Then n % 8 == 0, which fuses where K is long (bits straddle words, the last
# word is partial)
SHAPES = [(1, 64, 64), (17, 512, 64), (100, 1152, 192), (400, 64, 64), (784, 1216, 128),
          (1568, 128, 64), (49, 256, 256), (196, 512, 256), (100, 1152, 320), (7, 200, 1024),
          (50, 1152, 2048), (2047, 128, 256), (1000, 640, 512), (300, 72, 128),
          (1, 2560, 24), (33, 2560, 72), (100, 2560, 136), (777, 2560, 136), (260, 2600, 200),
          (1000, 4096, 264)]


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_few_tiles_bitmap(dt, shape):
    from paper_2511_19457_amd import abi
    tdt, dev = {"f16": torch.float16, "bf16": torch.bfloat16}[dt], torch.device("cuda")
    (m, k, n), seed = shape, 9700 + SHAPES.index(shape)
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(m, k, generator=g).relu_()
    x[m // 2:, : k // 2] = 0
    x[: m // 4] = 0                          # whole tiles without work, too
    w = torch.randn(n, k, generator=g) * k ** -0.5
    w[n // 2: n // 2 + 8] = 0                # zero blocks of y, and scattered zeros
    x, w = x.to(tdt).to(dev), w.to(tdt).to(dev)
    b = synth.normal((n,), dt, seed + 1)
    b[n // 2: n // 2 + 8] = 0
    b, r = b.to(dev), synth.normal((m, n), dt, seed + 2)
    r[:, n // 2: n // 2 + 8] = 0
    r = r.to(dev)
    d = abi.conv_desc(1, k, 1, m, n, 1, 1, dtype=tdt, has_bias=1)
    ws = torch.empty(max(16, abi.sparoa_conv2d_workspace_size(d, 0)), dtype=torch.uint8, device=dev)
    counts = torch.zeros(4, dtype=torch.int64, device=dev)
    mask = torch.zeros(abi.sparoa_mask_words(m, k, 1, 8), dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(x, m, k, 1, 8, 0, counts, mask)
    y = torch.full((m, n), float("nan"), dtype=tdt, device=dev)
    abi.sparoa_conv2d(d, abi.PATH_DENSE_MFMA, x, w, b, r, abi.ACT_RELU, None, y, ws)
    nb, words = m * (n // 8), abi.sparoa_mask_words(m, n, 1, 8)
    want_c = torch.zeros(4, dtype=torch.int64, device=dev)
    want_m = torch.zeros(words, dtype=torch.int32, device=dev)
    abi.sparoa_measure_sparsity(y, m, n, 1, 8, 0, want_c, want_m)
    path = torch.zeros(1, dtype=torch.int32, device=dev)
    for fill in (0, -1):
        for thr in (2.0, 0.0):      # routed dense, routed to skip
            for bitmap in (True, False):
                ym = torch.full_like(y, float("nan"))
                yc = torch.tensor([0, m * n, nb, nb], dtype=torch.int64, device=dev)
                ymask = torch.full((words + 2,), fill, dtype=torch.int32, device=dev)
                commit = torch.zeros(abi.COMMIT_WORDS_BYTES // 8, dtype=torch.int64, device=dev)
                abi.sparoa_conv2d_routed_measured(
                    d, thr, 0.0, abi.ROUTE_BLOCK, counts, x, w, b, r, abi.ACT_RELU, mask, ym, yc,
                    ymask[:words] if bitmap else None, ws, path, commit)
                torch.cuda.synchronize()
                what = (shape, dt, fill, thr, bitmap)
                assert torch.equal(y, ym) and torch.equal(yc, want_c), what
                assert not commit.any() and int(path.item()) == (thr == 0.0), what
                if bitmap:
                    assert torch.equal(ymask[:words], want_m), what
                    assert bool((ymask[words:] == fill).all()), what
