"""The row-per-pixel fp16 tiles with three and four ring slots (mid-size
grids) where their rings begin and end: windows of 1 to 6 stages of 64 taps
(fewer than, as many as and more than the slots, the last one partial),
pixel and channel counts off the tile, both operand types; every output
against the oracle, integer operands exact, and the same bits twice."""
import pytest
import torch

import oracle
import paper_2608_20725_amd as pkg
from gpu_util import Run, assert_kernel, check_full, say
from paper_2608_20725_amd import workloads

pytestmark = pytest.mark.gpu

TILES = ["c64p64s4", "c128p64s4", "c128p128s3w8", "c256p128s3w8"]
# K = 64, 72 (one tap group into stage 2), 192, 256, 328
SHAPES = [(1, 64, 9, 15, 72, 1, 1, 1), (2, 8, 11, 9, 260, 3, 3, 1), (1, 64, 5, 30, 130, 1, 3, 1),
          (3, 16, 7, 9, 40, 4, 4, 1), (1, 328, 12, 11, 96, 1, 1, 1)]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_deep_ring_tiles(shape, dtype, monkeypatch):
    N, Ci, H, W, Co, Kh, Kw, s = shape
    x, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 23)
    xi, wi = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 24, dist="int2")
    ref = torch.from_numpy(oracle.conv(xi.double().numpy(), wi.double().numpy(), s)).to(dtype)
    for tile in TILES:
        monkeypatch.setenv("IM2WIN_FP16_TILE", tile)
        assert_kernel(shape, dtype, "IM2WIN_FP16_TILE", tile)
        say("deep ring", tile, shape, dtype)
        r = Run(x, w, s, dtype)
        check_full(r, x, w)
        r.check_workspace_guard()
        r.check_out_guards()
        first = r.out.clone()
        r.rerun_conv()
        assert torch.equal(first.view(torch.int16), r.out.view(torch.int16))
        assert torch.equal(Run(xi, wi, s, dtype).out.cpu(), ref), tile


@pytest.mark.parametrize("shape,want", [
    ((24, 512, 9, 9, 512, 3, 3, 1), "c64p64s4"), ((128, 512, 7, 7, 512, 3, 3, 1), "c128p64s4"),
    ((32, 128, 30, 30, 128, 3, 3, 1), "c128p128s3w8"), ((128, 256, 56, 56, 256, 3, 3, 2), "c256p128s3w8"),
    ((128, 256, 14, 14, 256, 3, 3, 1), "k3c128p128t32s2"),
    # 144 channels: 64-channel rows where the busiest CU has less work with them (40 images, 543 / 815 tiles: 63.5 us
    # against 87.4), not at 32 (434 / 651: 51.8 against 50.8)
    ((40, 64, 62, 67, 144, 7, 7, 2), "c64p128s3"), ((32, 64, 62, 67, 144, 7, 7, 2), "c128p128s2"),
])
def test_mid_size_defaults(shape, want):
    assert pkg.conv_im2win_kernel_name(*shape, torch.float16).split()[1] == want
