"""A network's first 3x3 convolution fused with its 2x2 max pool: against the
CPU oracle and the two layers run separately, at sizes around the run of 32
windows that a wave takes at a time, and with more runs than waves."""
import numpy as np
import pytest

import oracle
from paper_2003_01538_amd import flexserve as fsb
from tests.test_gpu_kernels import BF16, assert_bf16_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,W", [(1, 2, 2), (2, 6, 16), (3, 10, 18), (1, 34, 14), (5, 18, 66), (1, 224, 224),
                                   (1, 2, 66), (1, 6, 42),   # 33 windows and 63: one and thirty-one in the last run
                                   (5, 202, 278)])           # 2194 runs: a second one a wave, whose step crosses rows and images
def test_first_conv_maxpool_fused(gpu_lib, B, H, W):
    rng = np.random.default_rng(H * 1000 + W)
    x = oracle.round_bf16(rng.standard_normal((B, H, W, 3)).astype(np.float32))
    w = oracle.round_bf16((rng.standard_normal((64, 3, 3, 3)) * np.sqrt(2.0 / 27)).astype(np.float32))
    b = (rng.standard_normal(64) * 0.1).astype(np.float32)
    g = fsb.fs_test_first_pool(x, w, b)
    c, ab = oracle.conv2d(x, w, b, 1, 1, 1, None, "bf16", want_abs=True)
    # the pooled value may be any window element that the sums' order brings to the top
    assert_bf16_close(g, oracle.maxpool(c, 2, 2, 0), oracle.maxpool(ab, 2, 2, 0), what=f"oracle {B}x{H}x{W}")
    sep = fsb.fs_test_maxpool(fsb.fs_test_conv(x, w, b, None, 1, 1, 1, BF16), 2, 2, 0, BF16)
    assert_bf16_close(g, sep, oracle.maxpool(ab, 2, 2, 0), what=f"two layers {B}x{H}x{W}")
    # infinities reach the same outputs, and a sum that is not a number leaves the ReLU as zero
    x[0, 0, 0, 0], x[-1, -1, -1, 1] = np.inf, -np.inf
    g = fsb.fs_test_first_pool(x, w, b)
    sep = fsb.fs_test_maxpool(fsb.fs_test_conv(x, w, b, None, 1, 1, 1, BF16), 2, 2, 0, BF16)
    assert np.array_equal(np.isinf(g), np.isinf(sep)) and not np.isnan(g).any() and np.isinf(g).any()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_a_pixel_reaches_only_the_windows_that_read_it(gpu_lib, value):
    # a pixel beside a window is read by one of its two columns of conv pixels:
    # the other column's sums stay finite and may be the window's maximum
    rng = np.random.default_rng(8)
    B, H, W = 2, 12, 20
    x = oracle.round_bf16(rng.standard_normal((B, H, W, 3)).astype(np.float32))
    w = oracle.round_bf16((rng.standard_normal((64, 3, 3, 3)) * np.sqrt(2.0 / 27)).astype(np.float32))
    b = (rng.standard_normal(64) * 0.1).astype(np.float32)
    _, ab = oracle.conv2d(x, w, b, 1, 1, 1, None, "bf16", want_abs=True)
    x[0, 3, 2, 0] = x[0, 8, 7, 1] = x[1, 0, 19, 2] = x[1, 11, 0, 0] = value
    g = fsb.fs_test_first_pool(x, w, b)
    sep = fsb.fs_test_maxpool(fsb.fs_test_conv(x, w, b, None, 1, 1, 1, BF16), 2, 2, 0, BF16)
    inf = np.isinf(sep)
    assert np.array_equal(np.isinf(g), inf) and not np.isnan(g).any()
    # the finite outputs as for finite inputs: the pixels' magnitudes are those of `ab` or drop out as a zero
    z = lambda v: np.where(inf, 0, v).astype(np.float32)
    assert_bf16_close(z(g), z(sep), oracle.maxpool(ab, 2, 2, 0), what=f"{value}")


def test_odd_maps_are_refused(gpu_lib):
    z = lambda *s: np.zeros(s, np.float32)
    for h, w in [(7, 8), (8, 7)]:
        with pytest.raises(fsb.FsError) as e:
            fsb.fs_test_first_pool(z(1, h, w, 3), z(64, 3, 3, 3), z(64))
        assert e.value.status == fsb.FS_ERR_UNSUPPORTED
