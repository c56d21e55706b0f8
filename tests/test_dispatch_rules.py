"""Kernel choice where the tile that suits most layers is behind: layers on
which a default once ran slower than the kernel it had replaced, each with the
kernel measured ahead (GPU time of the conv call, us, in the comments).  No
call here reaches a GPU."""
import os

import pytest

import paper_2608_20725_amd as pkg


@pytest.fixture(autouse=True)
def clean_env(monkeypatch):
    for v in [k for k in os.environ if k.startswith("IM2WIN_")]:
        monkeypatch.delenv(v)
    if not os.path.exists(pkg.library_path()):
        from paper_2608_20725_amd import build
        build.build()


def name(shape, dt, **kw):   # N, Ci, H, W, Co, Kh, Kw, s
    return pkg.conv_im2win_kernel_name(*shape, dt, **kw)


@pytest.mark.parametrize("shape,want", [
    # short windows: the tap-split tile's rounds cost more than its taps
    ((99, 3, 79, 79, 3, 3, 3, 1), "p4c8l8s2k16g4"),       # 68.1 tap-split, 38.2 with 192-pixel tiles
    ((71, 1, 115, 115, 10, 2, 2, 2), "p4c8l8s2k16g4"),    # 31.3, 17.3
    ((39, 17, 111, 111, 11, 1, 1, 1), "p4c8l8s2k16g4"),   # 59.8, 35.5
    ((125, 3, 111, 18, 3, 3, 1, 1), "p4c8l8s2k16g4"),     # 30.9, 15.7
    ((48, 3, 95, 95, 3, 2, 1, 2), "p4c8l8s2k16g4"),       # 17.4, 11.3
    # few tiles or longer windows: the tap-split tile
    ((1, 3, 230, 230, 64, 7, 7, 2), "p4c4l8s2k16g4t4"), ((4, 217, 28, 28, 63, 3, 3, 1), "p4c4l8s2k16g4t4"),
    ((1, 15, 37, 33, 223, 1, 1, 1), "p4c4l8s2k16g4t4"),
    ((2, 1, 55, 55, 509, 1, 1, 2), "p4c4l8s2k16g4t4"),    # 10.0 with p4c8l8s2k16g4, 8.6
    ((126, 1, 9, 9, 125, 3, 3, 1), "p4c4l8s2k16g4t4"),    # 10.0, 8.8
    # large grids
    ((32, 3, 230, 230, 64, 7, 7, 2), "p4c8l8s2k16g4"), ((128, 3, 227, 227, 64, 7, 7, 2), "p4c8l8s2k16g4"),
    ((128, 3, 227, 227, 96, 11, 11, 4), "p4c12l8s2k16g4"),
])
def test_dma32_unaligned(shape, want):
    assert name(shape, "f32") == "conv_fp32_dma " + want


@pytest.mark.parametrize("shape,want", [
    # windows shorter than a 128-tap stage
    ((17, 4, 57, 57, 43, 3, 3, 2), "p4c4l8s2k16t4"),      # 11.3 with p8c8l8s2k16t8w8, 9.9 p8c8l8s2k16t4, 8.1
    ((8, 8, 12, 38, 176, 1, 1, 1), "p4c4l8s2k16t4"), ((6, 8, 35, 35, 192, 7, 1, 2), "p4c4l8s2k16t4"),
    ((16, 256, 16, 16, 256, 3, 3, 1), "p8c8l8s2k16t8w8"),
])
def test_dma32_aligned_short_windows(shape, want):
    assert name(shape, "f32") == "conv_fp32_dma " + want


@pytest.mark.parametrize("shape,want", [
    # wide strided windows on few tiles, like any other few-tile layer
    ((2, 64, 28, 28, 64, 7, 7, 2), "p4c4l8s2k16t8w8"), ((1, 192, 19, 19, 11, 7, 7, 2), "p4c4l8s2k16t8w8"),
    ((8, 32, 60, 60, 15, 11, 11, 4), "p4c4l8s2k16t8w8"), ((24, 16, 33, 33, 40, 5, 5, 2), "p4c4l8s2k16t8w8"),
    ((2, 64, 28, 28, 64, 7, 7, 1), "p4c4l8s2k16t8w8"),
])
def test_dma32_wide_strided_windows(shape, want):
    assert name(shape, "f32") == "conv_fp32_dma " + want


def test_dma32_filter_range():
    """Filter offsets up to one stage past the window need 31 bits: a filter
    too long for 128-tap stages runs 64-tap ones, and the register-staged
    kernel only past those."""
    def at(Ci):
        return name((1, Ci, 2, 2, 16384, 1, 1, 1), "f32")
    assert at(32624) == "conv_fp32_dma p4c4l8s2k16t8w8"
    assert at(32688) == "conv_fp32_dma p4c8l8s2k16t4w8"
    assert at(32720).startswith("conv_fp32_kernel ")


@pytest.mark.parametrize("shape,want", [
    # short windows: a tap-split tile's first loads and final sum are not repaid
    ((112, 8, 13, 13, 128, 1, 1, 1), "c32p128s2"),        # 12.8 with c64p32s4t4, 9.3
    ((6, 8, 111, 45, 264, 2, 2, 2), "c32p128s2"),         # 10.1 with c32p32s2t4, 8.4
    ((10, 8, 24, 12, 288, 1, 1, 1), "c32p128s2"),         # 7.6 with c64p32s4t4, 6.8
    # longer ones, few pixels
    ((1, 256, 16, 16, 256, 3, 3, 1), "c32p32s4t4"), ((128, 512, 14, 14, 512, 3, 3, 1), "c32p128s2"),
    ((128, 64, 224, 224, 64, 7, 7, 2), "c64p128s2"),
])
def test_mfma32_short_windows(shape, want):
    assert name(shape, "f32", fp32_matrix_cores=True) == "conv_fp32_mfma " + want


@pytest.mark.parametrize("shape,want", [   # row-per-pixel tiles by their own number
    ((11, 536, 24, 20, 136, 7, 7, 1), "c64p64s4"),        # 158.2 with c64p128s3, 95.6
    ((20, 304, 35, 35, 184, 7, 7, 2), "c64p64s4"),
    ((16, 216, 41, 41, 176, 5, 5, 2), "c128p64s4"),       # 37.5 with c64p128s3, 33.0
    ((141, 32, 32, 38, 288, 11, 11, 4), "c64p128s3"),      # 32.8 with c128p128s3w8, 28.1
    ((144, 48, 14, 13, 184, 7, 3, 1), "c128p128s3w8"),    # 62.3 with c64p128s3, 44.8
    ((112, 64, 22, 18, 136, 5, 1, 1), "c64p128s3"),       # 568 tiles of 128 x 128, 852 of 64 x 128
    ((82, 504, 20, 20, 136, 5, 1, 1), "c128p128s2"),      # 410 and 615: 54.0 with c64p128s3, 46.8
])
def test_row_tiles_by_their_grid(shape, want, monkeypatch):
    monkeypatch.setenv("IM2WIN_FP16_KERNEL", "pipe")
    assert name(shape, "f16") == "conv_fp16_pipe " + want


@pytest.mark.parametrize("shape,want", [
    # long windows on two rounds of small-grid tiles
    ((18, 208, 24, 24, 344, 7, 7, 2), "conv_fp16_pipe c64p64s4"),     # 59.6 small-grid, 40.0
    ((4, 544, 72, 70, 96, 7, 7, 2), "conv_fp16_pipe c64p64s4"),       # 139.4, 85.8
    # two rounds of the smallest tile
    ((4, 112, 39, 39, 224, 7, 7, 2), "conv_fp16_direct c32p16w8"),    # 24.7 with c64p64s4, 20.5
    # where other kernels than that row tile would run
    ((5, 400, 21, 116, 4, 3, 3, 1), "conv_fp16_direct c32p32w8"),     # 29.9 column-staged, 16.2
    ((48, 136, 16, 16, 72, 7, 7, 1), "conv_fp16_direct c32p32w8"),    # 47.2 column-staged, 32.2
    # one round, or shorter windows
    ((1, 256, 16, 16, 256, 3, 3, 1), "conv_fp16_direct c32p16w8"), ((8, 512, 9, 9, 512, 3, 3, 1), "conv_fp16_direct c32p32w8"),
])
def test_direct_long_windows(shape, want):
    assert name(shape, "f16") == want


@pytest.mark.parametrize("shape,want", [
    # column slices half full of zeros (K_h*C_i of T_pad taps), many tiles
    ((43, 16, 106, 108, 200, 1, 3, 1), "conv_fp16_pipe c128p128s1"),  # 67.3 column-staged, 48.5
    ((39, 8, 87, 87, 240, 3, 3, 1), "conv_fp16_pipe c128p128s1"),     # 46.1, 40.0
    ((128, 64, 58, 58, 256, 3, 3, 1), "conv_fp16_col k3c128p128t32s2"),
    ((128, 256, 28, 28, 256, 3, 3, 1), "conv_fp16_col k3c128p128t32s2"),
])
def test_column_kernel_needs_filled_slices(shape, want):
    assert name(shape, "f16") == want


@pytest.mark.parametrize("shape,want", [
    # 3x3, up to 64 input and 65 to 128 output channels: by the grid, as any other layer
    ((1, 64, 16, 16, 128, 3, 3, 1), "conv_fp16_direct c32p16w8"), ((2, 64, 24, 24, 128, 3, 3, 1), "conv_fp16_direct c32p16w8"),
    ((5, 64, 30, 30, 128, 3, 3, 1), "conv_fp16_direct c64p32w8"), ((20, 64, 24, 24, 128, 3, 3, 1), "conv_fp16_pipe c128p64s4"),
    ((60, 64, 24, 24, 128, 3, 3, 1), "conv_fp16_pipe c128p128s3w8"), ((80, 64, 24, 24, 128, 3, 3, 1), "conv_fp16_col k3c128p128t32s2"),
])
def test_few_channels_by_grid(shape, want):
    assert name(shape, "f16") == want


@pytest.mark.parametrize("shape,want", [
    # strips of few pixels, long windows, many blocks a wave: a block's other lanes are idle
    ((27, 71, 26, 11, 672, 3, 3, 1), "conv_fp16_kernel c128p128u"),   # 42.2 one-wave, 26.8
    ((14, 13, 85, 15, 344, 7, 7, 1), "conv_fp16_kernel c128p128u"),   # 35.2, 24.9
    ((71, 73, 12, 12, 733, 3, 3, 1), "conv_fp16_kernel c128p128u"),   # 57.2, 40.9
    # few blocks, shorter windows, longer strips
    ((40, 71, 26, 11, 256, 3, 3, 1), "conv_fp16_seg w32"), ((27, 31, 26, 11, 672, 3, 3, 1), "conv_fp16_seg w96"),
    ((27, 71, 26, 18, 672, 3, 3, 1), "conv_fp16_seg w32"), ((128, 3, 227, 227, 96, 11, 11, 4), "conv_fp16_seg w96"),
])
def test_segment_waves_on_short_strips(shape, want):
    assert name(shape, "f16") == want


@pytest.mark.parametrize("shape,want", [
    # 256-row tiles only where C_o fills them
    ((31, 120, 53, 9, 520, 3, 3, 1), "c128p128s2"), ((23, 96, 19, 63, 289, 3, 3, 1), "c128p128s1"),
    ((128, 96, 24, 24, 256, 5, 5, 1), "c256p256s2w8"),
    # or where 128-channel tiles, storing single values, are not far fewer rounds ahead
    ((54, 40, 39, 37, 372, 2, 1, 2), "c256p256s2w8"),     # 23.8 with c128p128s2, 20.0
    ((51, 80, 22, 22, 388, 5, 5, 1), "c256p256s2w8"), ((51, 80, 22, 22, 392, 5, 5, 1), "c128p128s1"),
    ((51, 208, 22, 22, 388, 5, 5, 1), "c256p256s2w8"),
    ((51, 40, 22, 22, 268, 5, 5, 1), "c128p128s2"), ((51, 24, 22, 22, 268, 5, 5, 1), "c256p256s2w8"),
    ((78, 80, 22, 22, 392, 5, 5, 1), "c256p256s2w8"), ((78, 72, 22, 22, 392, 5, 5, 1), "c128p128s1"),
])
def test_wide_row_tiles_need_filled_rows(shape, want):
    assert name(shape, "f16") == "conv_fp16_pipe " + want


@pytest.mark.parametrize("shape,want", [
    ((23, 24, 34, 23, 532, 3, 3, 1), "k3c256p192t32s2w8"),     # 33.2 with k3c128p128t32s2, 24.1
    ((105, 16, 19, 19, 308, 3, 3, 1), "k3c256p256t32s2w8"),    # 29.8, 22.0
    ((23, 376, 34, 23, 532, 3, 3, 1), "k3c256p192t32s2w8"),
    ((105, 16, 24, 24, 188, 3, 3, 1), "k3c256p256t32s2w8"),
    ((23, 24, 34, 23, 536, 3, 3, 1), "k3c128p128t32s2"), ((23, 24, 34, 23, 534, 3, 3, 1), "k3c128p128t32s2"),
])
def test_wide_column_tiles_on_8_byte_rows(shape, want):
    assert name(shape, "f16") == "conv_fp16_col " + want
