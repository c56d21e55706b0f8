"""Small-grid 16-bit kernel (conv_fp16_direct: taps split over the waves of a
workgroup, operands straight to registers, the caller's filter read without a
pack) against the oracle, at the sizes where its tiles, its 32-tap steps and
its channel groups end: windows of one tap group, of a whole number of steps
and one element more, fewer steps than waves, odd and single-group channel
counts, one pixel, dilation and stride, infinities outside the window of the
last step.  Bars: the fp16 and bf16 ones of the other kernels (one output
rounding plus K * 2^-24 of fp32 accumulation)."""
import pytest
import torch

import oracle
import paper_2608_20725_amd as pkg
from gpu_util import Run, check_full, say
from paper_2608_20725_amd import workloads

pytestmark = pytest.mark.gpu

VARIANTS = ["c32p16w8", "c32p32w8", "c64p32w8", "c64p64w8", "c64p64w4"]

SHAPES = [  # N, Ci, H, W, Co, Kh, Kw, s
    (1, 8, 1, 1, 2, 1, 1, 1),        # one pixel, one tap group, two channels
    (1, 32, 4, 5, 4, 1, 1, 1),       # exactly one step
    (1, 33, 5, 4, 64, 1, 1, 1),      # one element past a step, unaligned windows
    (2, 24, 6, 9, 68, 3, 2, 1),      # K % 32 = 16; one pixel past a 64-pixel tile: 2*4*8
    (1, 5, 9, 13, 33, 3, 5, 2),      # odd C_i and C_o
    (3, 64, 9, 9, 132, 3, 3, 1),     # 18 steps: more than two batches of eight waves for some
    (2, 7, 11, 10, 35, 7, 7, 3),     # windows crossing filter rows inside a lane's eight taps
    (1, 520, 3, 3, 96, 3, 3, 1),     # 147 steps, one pixel
]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_direct_edges(monkeypatch, shape, dtype):
    N, Ci, H, W, Co, Kh, Kw, s = shape
    x, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 77)
    for v in VARIANTS:
        monkeypatch.setenv("IM2WIN_FP16_DIRECT", v)
        if v.startswith("c64") and Co % 4:
            with pytest.raises(pkg.Im2winError):
                pkg.conv_im2win_kernel_name(N, Ci, H, W, Co, Kh, Kw, s, dtype)
            continue
        assert pkg.conv_im2win_kernel_name(N, Ci, H, W, Co, Kh, Kw, s, dtype) == "conv_fp16_direct " + v
        say("direct", shape, dtype, v)
        r = Run(x, w, s, dtype)
        r.check_workspace_guard()
        r.check_out_guards()
        check_full(r, x, w)
        first = r.out.clone()
        r.rerun_conv()
        assert torch.equal(first.view(torch.int16), r.out.view(torch.int16))


def test_direct_integers_exact(monkeypatch):
    """Integer operands: every partial sum is exact, so any split of the taps gives the same bits."""
    x, w = workloads.draw(2, 20, 9, 11, 44, 3, 3, 5, dist="int2")
    ref = oracle.conv(x.double().numpy(), w.double().numpy(), 1)
    for v in VARIANTS:
        monkeypatch.setenv("IM2WIN_FP16_DIRECT", v)
        r = Run(x, w, 1, torch.float16)
        assert torch.equal(r.out.cpu(), torch.from_numpy(ref).half()), v


@pytest.mark.parametrize("Ci", [8, 9])
def test_direct_last_step_ignores_next_window(monkeypatch, Ci):
    """The last step's taps past K read the next window's column and rows past
    the filter: an infinity there must not reach a pixel whose window does not hold it."""
    x, w = workloads.draw(1, Ci, 6, 12, 16, 3, 3, 9)
    x[:, :, 6:, :] = float("inf")
    ref = oracle.conv(x[:, :, :6, :].double().half().double().numpy(), w.half().double().numpy(), 1)
    for v in VARIANTS:
        monkeypatch.setenv("IM2WIN_FP16_DIRECT", v)
        r = Run(x, w, 1, torch.float16)
        got = r.out[:, :, :4, :].double().cpu()
        assert torch.isfinite(got).all(), v
        assert (got - torch.from_numpy(ref)).abs().max() < 0.05
        assert not torch.isfinite(r.out[:, :, 4:, :]).any()


@pytest.mark.parametrize("d,pad,Ci,Co", [(2, 2, 16, 64), (3, 0, 9, 33)])
def test_direct_dilated_default(d, pad, Ci, Co):
    """Dilated small layers take this kernel by default."""
    N, H, W, K = 2, 13, 15, 3
    x, w = workloads.draw(N, Ci, H, W, Co, K, K, 3)
    dt = torch.float16
    Hp, Wp = H + 2 * pad, W + 2 * pad
    assert pkg.conv_im2win_kernel_name(N, Ci, Hp, Wp, Co, K, K, 1, dt, dilation=d).startswith("conv_fp16_direct ")
    xd, wd = x.to(dt).cuda(), w.to(dt).cuda()
    Ho, Wo = pkg.conv_output_dims_dilated(Hp, Wp, K, K, 1, d)
    ws = torch.empty(pkg.conv_workspace_bytes_dilated(N, Ci, Hp, Wp, Co, K, K, 1, d, dt), dtype=torch.uint8,
                     device="cuda")
    out = torch.empty((N, Ho, Wo, Co), dtype=dt, device="cuda")
    pkg.conv_im2win_transform_dilated(xd, ws, Co, K, K, 1, pad, pad, d)
    pkg.conv_im2win_dilated(ws, wd, out, N, Ci, Hp, Wp, 1, d)
    ref = torch.nn.functional.conv2d(xd.cpu().double().permute(0, 3, 1, 2), wd.cpu().double().permute(3, 2, 0, 1),
                                     padding=pad, dilation=d).permute(0, 2, 3, 1)
    # |x|, |w| <= 1: one fp16 rounding of |y| <= K plus the accumulation
    assert (out.cpu().double() - ref).abs().max() <= 2.0 ** -11 * ref.abs().max() + 1e-3
