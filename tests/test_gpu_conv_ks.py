"""The convolution kernel for layers with few output tiles (the reduction
split over a workgroup's waves): every tile of it against the CPU oracle and
against the general kernels at the sizes where it can go wrong, its two weight
routes against each other, and its projection shortcut layer by layer."""
import numpy as np
import pytest

import oracle
import workloads as wl
from paper_2003_01538_amd import flexserve as fsb
from tests.test_gpu_kernels import BF16, _conv_inputs, assert_bf16_close
from tests.test_gpu_layers import check_layers
from tests.test_zz_no_alloc import _run as noalloc_equals_test_conv

pytestmark = pytest.mark.gpu

CASES = [
    # B, H, W, Cin, Cout, k, stride, pad, relu, residual
    (1, 1, 1, 512, 128, 3, 1, 1, 1, 1),     # one pixel: every tap but the centre reads the row of zeros
    (1, 3, 2, 64, 32, 3, 1, 1, 0, 0),       # one channel block, nine K-tiles over eight waves
    (1, 4, 8, 128, 128, 3, 1, 1, 1, 0),     # exactly one 32-pixel tile
    (1, 3, 11, 128, 64, 3, 1, 1, 1, 1),     # 33 pixels: a second tile of one pixel
    (3, 5, 13, 64, 128, 3, 1, 1, 1, 1),     # tiles across rows and images, ragged M
    (2, 7, 7, 512, 512, 3, 1, 1, 1, 1),     # the largest input in LDS
    (5, 15, 13, 256, 128, 3, 2, 1, 1, 0),   # stride 2, odd map: images of odd length
    (2, 14, 14, 128, 256, 3, 2, 1, 0, 1),   # stride 2, even map, residual
    (1, 2, 2, 64, 128, 3, 2, 1, 1, 0),      # stride 2 down to one pixel
    (1, 9, 70, 64, 64, 3, 1, 1, 1, 1),      # rows longer than a tile
    (2, 9, 9, 512, 128, 1, 1, 0, 1, 1),     # 1x1: the tile's own pixels
    (2, 9, 9, 1024, 96, 1, 2, 0, 0, 0),     # 1x1 stride 2, three channel blocks
]


@pytest.mark.parametrize("ci", range(len(CASES)))
def test_every_tile_matches_the_oracle_and_the_general_kernels(gpu_lib, ci):
    case = CASES[ci]
    x, w, b, r = _conv_inputs(case, BF16, 300 + ci)
    s, p, relu = case[6:9]
    o, ab = oracle.conv2d(x, w, b, s, p, relu, r, "bf16", want_abs=True)
    ran = {}
    for t in list(range(fsb.fs_conv_num_tiles(BF16))) + [-1]:
        name = fsb.fs_conv_tile_name(BF16, t) if t >= 0 else "auto"
        if not ("ks_" in name or "dma2_64x128" in name or t < 0):
            continue
        try:
            g = fsb.fs_test_conv(x, w, b, r, s, p, relu, BF16, tile=t)
        except fsb.FsError as e:  # Cout not a multiple of the tile's, fewer K-tiles than waves, input too large for LDS
            assert e.status == fsb.FS_ERR_UNSUPPORTED and t >= 0
            continue
        ran[name] = g
        # one bf16 ulp plus the fp32 sums' order (2^-16 of the summed magnitudes), as for every conv tile
        assert_bf16_close(g, o, ab, what=f"case {ci} {name}")
    assert "bf16dma2_64x128_w4_v8" in ran and sum("ks_" in n for n in ran) >= 1, list(ran)
    # few tiles: the automatic choice is this kernel, bit for bit one of its tiles
    assert any(np.array_equal(ran["auto"].view(np.uint32), g.view(np.uint32)) for n, g in ran.items() if "ks_" in n)


@pytest.mark.parametrize("case", [(1, 7, 7, 512, 512, 3, 1, 1, 1, True), (7, 7, 7, 512, 512, 3, 1, 1, 1, True),
                                  (13, 7, 7, 512, 512, 3, 1, 1, 0, False), (5, 15, 13, 256, 512, 3, 2, 1, 1, False),
                                  (9, 28, 28, 128, 256, 3, 2, 1, 1, False), (8, 28, 28, 128, 128, 3, 1, 1, 1, True),
                                  (3, 14, 14, 1024, 256, 1, 1, 0, 1, False), (7, 14, 14, 256, 512, 3, 2, 1, 1, False),
                                  (2, 7, 7, 2048, 512, 1, 1, 0, 1, False), (1, 56, 56, 64, 64, 3, 1, 1, 1, True)])
def test_packed_and_fragment_ordered_weights_give_the_same_bits(gpu_lib, case):
    # fs_test_conv has the fragment-ordered copy, the allocation-free entry point only the packed rows
    noalloc_equals_test_conv(*case, seed=5)


@pytest.mark.parametrize("B", [1, 3, 7])
def test_every_layer_of_a_small_batch(B):
    # projection shortcuts included: their rows, weights and summed biases
    models = [wl.build_model("resnet18", 2001), wl.build_model("resnet18", 2002)]
    imgs = wl.images_ragged(70 + B, B, 200, 260)
    prepared = [oracle.prepare_model(m, "bf16") for m in models]
    with fsb.Ensemble(models, (224, 224), wl.IMAGENET_MEAN, wl.IMAGENET_STD, "bf16", max_batch=8) as ens:
        fsb.fs_debug_capture(ens.handle, B - 1)
        first = ens.infer(imgs)
        again = ens.infer(imgs)
        for k in ("logits", "probs", "vote", "top1"):
            assert np.array_equal(first[k], again[k]), k
        for m, layers in enumerate(models):
            check_layers(ens, layers, prepared[m], "bf16", imgs, B - 1, m, (224, 224), [])
        fsb.fs_debug_capture(ens.handle, -1)
