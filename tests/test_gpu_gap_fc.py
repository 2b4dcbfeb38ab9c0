"""The global average pool and the classifier in one launch: the pooled
tensor bit-equal to the pool's own launch, the outputs to the classifier's
(bf16, the same matrix steps in the same order) or within the fp32 bound of
any order of the sum."""
import numpy as np
import pytest

import oracle
from paper_2003_01538_amd import flexserve as fsb
from tests.test_gpu_kernels import BF16, F32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [BF16, F32])
@pytest.mark.parametrize("B,H,W,K,N,relu", [
    (1, 7, 7, 512, 1000, 0),   # the largest K
    (4, 16, 16, 32, 10, 0),    # one matrix step, fewer features than a wave takes
    (7, 7, 7, 512, 1000, 1),
    (32, 7, 7, 512, 65, 0),    # one feature in the second workgroup
    (2, 17, 17, 64, 33, 1),    # the most channels of the fp32 kernel for few, more pixels than one round
    (2, 3, 3, 128, 33, 0),     # ... of the bf16 one
    (2, 1, 1, 8, 1, 0),        # one pixel, one vector of channels
    (3, 5, 3, 264, 100, 0),    # fewer pixels than pixel lanes, K no multiple of a step
])
def test_one_launch_equals_two(gpu_lib, prec, B, H, W, K, N, relu):
    rng = np.random.default_rng(B * 7 + K)
    x = rng.standard_normal((B, H, W, K)).astype(np.float32)
    w = (rng.standard_normal((N, K)) * np.sqrt(2.0 / K)).astype(np.float32)
    b = (rng.standard_normal(N) * 0.1).astype(np.float32)
    if prec == BF16:
        x, w = oracle.round_bf16(x), oracle.round_bf16(w)
    pooled, y = fsb.fs_test_gap_fc(x, w, b, relu, prec)
    assert np.array_equal(pooled.view(np.uint32), fsb.fs_test_gap(x, prec).reshape(B, K).view(np.uint32))
    two = fsb.fs_test_fc(pooled, w, b, relu, prec)
    if prec == BF16:
        assert np.array_equal(y.view(np.uint32), two.view(np.uint32))
    ab = np.abs(pooled).astype(np.float64) @ np.abs(w).astype(np.float64).T
    o = oracle.fc(pooled, w, b, relu, "fp32")
    assert np.all(np.abs(y - o) <= 1e-5 * ab + 1e-6), np.abs(y - o).max()  # as for the layer by itself


def test_what_runs_as_two(gpu_lib):
    z = lambda *s: np.zeros(s, np.float32)
    for B, H, K, N in [(1, 7, 520, 10), (1, 9, 512, 10), (64, 7, 512, 1000)]:
        with pytest.raises(fsb.FsError) as e:
            fsb.fs_test_gap_fc(z(B, H, H, K), z(N, K), z(N), 0, BF16)
        assert e.value.status == fsb.FS_ERR_UNSUPPORTED
