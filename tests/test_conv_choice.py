"""Which kernel a convolution layer gets where nothing is timed: layers that
were measured, on both sides of each rule's line.  The rules see shapes only,
so this needs no GPU."""
import re

import pytest

from paper_2003_01538_amd import flexserve as fsb


def tile_size(name):
    return tuple(int(v) for v in re.search(r"_(\d+)x(\d+)", name).groups())


@pytest.mark.parametrize("cin,cout,k,hw,B,Z", [
    (3, 16, 3, 32, 8, 3), (3, 16, 3, 32, 64, 1), (3, 16, 3, 32, 64, 3),   # a small net's first layer
    (64, 24, 1, 32, 64, 2), (32, 8, 1, 56, 64, 2), (3, 32, 3, 56, 8, 3), (32, 96, 3, 56, 4, 2),
])
def test_fp32_layers_do_not_run_on_half_empty_tiles(cin, cout, k, hw, B, Z):
    name, split = fsb.fs_test_conv_choice(B, hw, hw, cin, cout, k, 1, k // 2, fsb.FS_F32, Z)
    bm, bn = tile_size(name)
    assert bn == 32 and split == 1, name


@pytest.mark.parametrize("cin,cout,hw,B,Z,want", [
    (64, 64, 56, 8, 3, "f32_64x64_v4"), (256, 256, 14, 8, 3, "f32_32x32_k4_v4"), (512, 512, 7, 1, 3, "f32_32x32_k8_v4"),
])
def test_fp32_layers_whose_channels_fill_the_tile(cin, cout, hw, B, Z, want):
    assert fsb.fs_test_conv_choice(B, hw, hw, cin, cout, 3, 1, 1, fsb.FS_F32, Z) == (want, 1)


def test_fp32_filters_of_any_size_have_a_kernel():
    # a reduction of 2^24 values was refused while the kernel's index arithmetic had no form for it
    assert fsb.fs_test_conv_choice(1, 2048, 2048, 4, 8, 2048, 1, 0, fsb.FS_F32)[1] == 1


# Layers whose reduction could be split over a workgroup's waves, and the kernel that was measured faster.
@pytest.mark.parametrize("B,hw,cin,cout,k,stride,Z,packed,residual,split", [
    (1, 7, 512, 512, 3, 1, 3, False, True, True),       # few tiles: 7.3 us against 26.3
    (8, 28, 128, 256, 3, 2, 1, False, False, True),     # ... and a split over workgroups saved: 9.3 against 16.9
    (8, 28, 128, 256, 3, 2, 1, True, False, True),
    (1, 7, 512, 512, 3, 1, 1, True, True, True),
    (1, 28, 128, 512, 1, 1, 2, False, True, False),     # two K-tiles: 5.3 us against 4.4
    (4, 12, 128, 384, 1, 2, 1, False, False, False),
    (12, 14, 512, 512, 3, 1, 5, False, False, False),   # three rounds of one workgroup a CU: 64 us against 51
    (7, 28, 512, 512, 3, 1, 2, False, False, False),    # 63 us against 51
    (6, 16, 2048, 512, 1, 1, 2, False, True, False),    # 29 us against 22
    (19, 28, 512, 128, 1, 1, 1, True, False, False),    # eight K-tiles: 8.6 us against 7.9
    (12, 31, 512, 512, 3, 1, 1, True, False, False),    # packed rows that find no LDS to be turned in: 109 us against 67
    (10, 28, 512, 512, 3, 1, 1, True, False, False),    # 73 us against 40
    (4, 28, 512, 512, 3, 1, 1, True, False, False),     # 37 us against 34
    (20, 17, 512, 512, 3, 1, 1, True, False, False),    # 39 us against 35
])
def test_the_split_reduction_kernel_takes_the_layers_it_is_faster_on(B, hw, cin, cout, k, stride, Z, packed, residual,
                                                                     split):
    name, _ = fsb.fs_test_conv_choice(B, hw, hw, cin, cout, k, stride, k // 2, fsb.FS_BF16, Z, packed, residual)
    assert ("ks_" in name) == split, name


def test_the_allocation_free_call_costs_a_split_layer_as_it_runs():
    # in four splits: 64x128 tiles 20.0 us, 64x64, the choice for the unsplit layer, 21.0
    assert fsb.fs_test_conv_choice(25, 7, 10, 2048, 512, 1, 1, 0, fsb.FS_BF16, 1, packed=True) == \
        ("bf16dma2_64x128_w4_v8", 4)


def test_the_allocation_free_call_accepts_by_its_scratch():
    # few tiles, so that no partial sums would be written; what is accepted does not follow the kernel
    with pytest.raises(fsb.FsError) as e:
        fsb.fs_test_conv_choice(5, 16, 16, 256, 1216, 3, 1, 1, fsb.FS_BF16, 1, packed=True)
    assert e.value.status == fsb.FS_ERR_UNSUPPORTED
    assert fsb.fs_test_conv_choice(5, 16, 16, 256, 1216, 3, 1, 1, fsb.FS_BF16, 1)[0]


@pytest.mark.parametrize("B,hw,packed", [(24, 16, True), (32, 14, False)])
def test_of_nearly_equal_tiles_the_larger_one(B, hw, packed):
    name, _ = fsb.fs_test_conv_choice(B, hw, hw, 256, 256, 3, 1, 1, fsb.FS_BF16, 1, packed)
    assert name == "bf16ks_64x128_w8_v8", name
