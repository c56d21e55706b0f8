"""The tap-split fp32 tiles of small grids (32 x 32 and 64 x 64 pixels x
channels, 64 or 128 taps per stage, 16- and 4-byte window loads) against the
oracle: windows shorter than a stage, of whole stages and one granule more,
pixel and channel counts off the tile, C_o not a multiple of 4; integers exact
and the same bits twice."""
import pytest
import torch

import oracle
import paper_2608_20725_amd as pkg
from gpu_util import Run, assert_kernel, check_full, say
from paper_2608_20725_amd import workloads

pytestmark = pytest.mark.gpu

ALIGNED = ["p4c4l8s2k16t4", "p4c4l8s2k16t8w8", "p8c8l8s2k16t8w8"]
UNALIGNED = ["p4c4l8s2k16g4t4", "p4c8l8s2k16g4t4w8"]
SHAPES = [  # N, Ci, H, W, Co, Kh, Kw, s
    (1, 4, 1, 1, 4, 1, 1, 1), (1, 128, 5, 7, 33, 1, 1, 1), (2, 132, 4, 9, 66, 1, 1, 1),
    (2, 32, 11, 12, 100, 3, 3, 2), (1, 16, 10, 9, 7, 4, 4, 1), (3, 64, 9, 9, 31, 3, 3, 1),
]
ODD = [(1, 1, 1, 1, 3, 1, 1, 1), (1, 65, 5, 7, 33, 1, 1, 1), (2, 3, 21, 23, 96, 11, 11, 4),
       (2, 7, 9, 14, 40, 3, 5, 1), (3, 21, 6, 6, 65, 3, 3, 1)]


@pytest.mark.parametrize("shape,names", [(s, ALIGNED + UNALIGNED) for s in SHAPES] + [(s, UNALIGNED) for s in ODD],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else "")
def test_small_grid_tiles(shape, names, monkeypatch):
    N, Ci, H, W, Co, Kh, Kw, s = shape
    x, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 51)
    xi, wi = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 52, dist="int2")
    ref = torch.from_numpy(oracle.conv(xi.double().numpy(), wi.double().numpy(), s)).float()
    for name in names:
        monkeypatch.setenv("IM2WIN_FP32_KERNEL", name)
        assert_kernel(shape, torch.float32, "IM2WIN_FP32_KERNEL", name)
        say("fp32 small", name, shape)
        r = Run(x, w, s, torch.float32)
        check_full(r, x, w)
        r.check_workspace_guard()
        r.check_out_guards()
        first = r.out.clone()
        r.rerun_conv()
        assert torch.equal(first.view(torch.int32), r.out.view(torch.int32))
        assert torch.equal(Run(xi, wi, s, torch.float32).out.cpu(), ref), name


@pytest.mark.parametrize("shape,want", [
    ((1, 256, 16, 16, 256, 3, 3, 1), "p4c4l8s2k16t8w8"), ((6, 32, 30, 30, 48, 1, 1, 1), "p4c4l8s2k16t4"),
    ((16, 256, 16, 16, 256, 3, 3, 1), "p8c8l8s2k16t8w8"), ((128, 512, 7, 7, 512, 3, 3, 1), "p4c8l8s2k16t4w8"),
    ((1, 3, 230, 230, 64, 7, 7, 2), "p4c4l8s2k16g4t4"), ((32, 3, 230, 230, 64, 7, 7, 2), "p4c8l8s2k16g4"),
])
def test_small_grid_defaults(shape, want):
    assert pkg.conv_im2win_kernel_name(*shape, torch.float32).split()[1] == want


@pytest.mark.parametrize("shape", [(1, 4, 1, 1, 4, 1, 1, 1), (1, 32, 5, 7, 33, 1, 1, 1), (2, 36, 4, 9, 66, 1, 1, 1),
                                   (2, 32, 11, 12, 100, 3, 3, 2), (3, 64, 9, 9, 31, 3, 3, 1), (1, 20, 9, 8, 7, 5, 5, 2)],
                         ids=lambda v: "x".join(map(str, v)))
def test_matrix_core_tap_split_tiles(shape, monkeypatch):
    """fp32 on the matrix cores, the taps of a stage split over four waves:
    windows of one chunk, one stage, and one chunk into a stage."""
    N, Ci, H, W, Co, Kh, Kw, s = shape
    x, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 61)
    xi, wi = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 62, dist="int2")
    ref = torch.from_numpy(oracle.conv(xi.double().numpy(), wi.double().numpy(), s)).float()

    def conv(a, b):
        r = Run(a, b, s, torch.float32, conv=False)
        pkg.conv_im2win_fp32_mfma(r.ws, r.wd, r.out, r.N, r.Ci, r.H, r.W, s)
        torch.cuda.synchronize()
        return r

    for name in ("c32p32s4t4", "c32p32s2t4", "c64p32s4t4"):
        monkeypatch.setenv("IM2WIN_FP32_MFMA_TILE", name)
        assert pkg.conv_im2win_kernel_name(*shape, "f32", fp32_matrix_cores=True) == "conv_fp32_mfma " + name
        say("fp32 mfma split", name, shape)
        r = conv(x, w)
        check_full(r, x, w)
        r.check_workspace_guard()
        r.check_out_guards()
        assert torch.equal(r.out.view(torch.int32), conv(x, w).out.view(torch.int32))
        assert torch.equal(conv(xi, wi).out.cpu(), ref), name
