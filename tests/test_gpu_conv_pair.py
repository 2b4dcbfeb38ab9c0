"""The widening and the narrowing 1x1 convolution in one launch: both outputs
bit-equal to the two launches they replace, for every channel combination the
kernel takes, and the two launches themselves against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2003_01538_amd import flexserve as fsb
from tests.test_gpu_kernels import assert_bf16_close

pytestmark = pytest.mark.gpu

# channels in, of the shortcut's input, of the wide tensor, out
CHANNELS = [(64, 64, 256, 64), (64, 0, 256, 64), (64, 0, 256, 128), (128, 256, 512, 128), (128, 0, 512, 128),
            (128, 0, 512, 256), (256, 0, 1024, 256), (64, 0, 128, 64), (128, 0, 1024, 128)]


@pytest.mark.parametrize("c", CHANNELS)
@pytest.mark.parametrize("B,H,W,stride2", [(1, 1, 1, 1), (1, 4, 8, 2), (3, 5, 11, 2), (1, 16, 24, 1), (2, 14, 14, 2)])
def test_one_launch_equals_two(gpu_lib, c, B, H, W, stride2):
    # one pixel; one wave's 32; a ragged 165; three whole workgroups; 392
    cin, cin2, n1, n2 = c
    rng = np.random.default_rng(cin + n1 + n2 + H)
    g = lambda *s, k=1.0: oracle.round_bf16((rng.standard_normal(s) * k).astype(np.float32))
    x = g(B, H, W, cin)
    x2 = g(B, (H - 1) * stride2 + 2, (W - 1) * stride2 + 1, cin2) if cin2 else None
    w1, w2 = g(n1, cin + cin2, k=(cin + cin2) ** -0.5), g(n2, n1, k=n1 ** -0.5)
    b1, b2 = g(n1), g(n2)
    for res in ([None] if cin2 else [g(B, H, W, n1), None]):
        y, t = fsb.fs_test_conv_pair(x, x2, stride2, w1, b1, res, w2, b2, True)
        ys, ts = fsb.fs_test_conv_pair(x, x2, stride2, w1, b1, res, w2, b2, False)
        assert np.array_equal(y.view(np.uint32), ys.view(np.uint32)), c
        assert np.array_equal(t.view(np.uint32), ts.view(np.uint32)), c
        xx = x if x2 is None else np.concatenate([x, x2[:, : (H - 1) * stride2 + 1 : stride2, ::stride2]], axis=3)
        o, ab = oracle.conv2d(xx, w1[:, None, None, :], b1, 1, 0, 1, res, "bf16", want_abs=True)
        assert_bf16_close(y, o, ab, what=f"wide {c}")
        o, ab = oracle.conv2d(y, w2[:, None, None, :], b2, 1, 0, 1, None, "bf16", want_abs=True)
        assert_bf16_close(t, o, ab, what=f"narrow {c}")


def test_refused_shapes(gpu_lib):
    z = lambda *s: np.zeros(s, np.float32)
    for cin, n1, n2 in [(192, 256, 64), (64, 192, 64), (64, 256, 96), (64, 2048, 64)]:
        with pytest.raises(fsb.FsError) as e:
            fsb.fs_test_conv_pair(z(1, 2, 2, cin), None, 1, z(n1, cin), z(n1), None, z(n2, n1), z(n2), True)
        assert e.value.status == fsb.FS_ERR_UNSUPPORTED
