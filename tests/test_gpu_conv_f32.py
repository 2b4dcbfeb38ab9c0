"""The fp32 convolution kernel: every tile against the CPU oracle at the sizes
where it can go wrong (tile edges, channel counts whose K-tiles lie in one
filter tap and such that do not, reductions shorter than the waves that split
them)."""
import numpy as np
import pytest

import oracle
from paper_2003_01538_amd import flexserve as fsb
from tests.test_gpu_kernels import F32, _conv_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, W, Cin, Cout, k, stride, pad, relu, residual
    (1, 1, 1, 32, 8, 1, 1, 0, 1, 1),      # one pixel, one K-tile over up to eight waves
    (1, 5, 13, 3, 16, 3, 1, 1, 1, 0),     # padded first layer, 65 pixels, half a channel block
    (2, 33, 31, 3, 24, 7, 2, 3, 1, 0),    # 7x7 on odd maps: taps past the filter in the last K-tile
    (1, 9, 7, 24, 40, 3, 1, 1, 0, 1),     # K-tiles across taps (24 channels), a ragged channel block
    (1, 8, 8, 48, 32, 5, 1, 2, 1, 1),     # ... with 48 channels and a 5x5 filter
    (3, 7, 7, 64, 72, 3, 1, 1, 1, 1),     # tiles across images, a channel block of 8
    (1, 8, 8, 32, 64, 3, 2, 1, 1, 0),     # Kp > K, stride 2
    (2, 6, 10, 96, 32, 1, 2, 0, 0, 1),    # 1x1 stride 2
    (1, 4, 4, 256, 64, 3, 1, 1, 1, 0),    # a long reduction on few pixels
    (1, 6, 6, 64, 32, 3, 3, 0, 1, 0),     # stride 3 without padding
]


@pytest.mark.parametrize("ci", range(len(CASES)))
def test_every_tile_matches_the_oracle(gpu_lib, ci):
    case = CASES[ci]
    x, w, b, r = _conv_inputs(case, F32, 500 + ci)
    s, p, relu = case[6:9]
    o, ab = oracle.conv2d(x, w, b, s, p, relu, r, "fp32", want_abs=True)
    for t in list(range(fsb.fs_conv_num_tiles(F32))) + [-1]:
        g = fsb.fs_test_conv(x, w, b, r, s, p, relu, F32, tile=t)
        # fp32 sums in another order than the oracle's double sums, as for every fp32 conv
        assert np.all(np.abs(g - o) <= 1e-5 * ab + 1e-6), (ci, t, np.abs(g - o).max())
        assert np.array_equal(g, fsb.fs_test_conv(x, w, b, r, s, p, relu, F32, tile=t)), (ci, t)


@pytest.mark.parametrize("H,W,k,stride", [
    (3, 1 << 22, 3, 1 << 16),   # a filter that spans 3 x 2^22 pixels: row * width needs more than 24 bits
    (2048, 2048, 2048, 1),      # a reduction of 2^24 stored values
])
def test_filters_beyond_24_bit_arithmetic(gpu_lib, H, W, k, stride):
    rng = np.random.default_rng(k)
    x = rng.standard_normal((1, H, W, 3), np.float32)
    w = rng.standard_normal((8, k, k, 3), np.float32)
    b = rng.standard_normal(8).astype(np.float32)
    o, ab = oracle.conv2d(x, w, b, stride, 0, 0, None, "fp32", want_abs=True)
    g = fsb.fs_test_conv(x, w, b, None, stride, 0, 0, F32)
    assert np.all(np.abs(g - o) <= 1e-5 * ab + 1e-6), np.abs(g - o).max()
