"""The one-wave segment kernel (filter kept in LDS, each wave 32 pixels of one
strip) against the oracle where its pieces end: pixel starts on 8-, 4- and
2-byte boundaries, windows of one 16-tap step, of whole steps and one element
more, strips of fewer than, exactly and just over 32 pixels, channel counts
off 8, 32 and odd, several channel groups, single pixels; infinities that
start right after a pixel's window; integers exact."""
import pytest
import torch

import oracle
import paper_2608_20725_amd as pkg
from gpu_util import Run, assert_kernel, check_full, say
from paper_2608_20725_amd import workloads

pytestmark = pytest.mark.gpu

VARIANTS = ["w32", "w64", "w96", "w128"]
SHAPES = [  # N, Ci, H, W, Co, Kh, Kw, s
    (1, 3, 32, 34, 32, 3, 3, 1),      # 2-byte starts (S = 9), 32 pixels per strip, two steps
    (2, 3, 23, 73, 64, 7, 7, 2),      # 4-byte starts (S = 42), 34 pixels per strip
    (2, 3, 23, 40, 96, 11, 11, 4),    # 8-byte starts (S = 132), 8 pixels per strip
    (3, 1, 5, 40, 5, 1, 1, 1),        # one tap, odd C_o
    (1, 4, 6, 35, 33, 2, 2, 1),       # K = 16: one whole step; one channel past a group
    (1, 17, 4, 33, 40, 1, 1, 1),      # K = 17: one element into the second step
    (2, 12, 9, 9, 100, 3, 5, 2),      # C_o % 4 = 0, several groups of 32 and 64
    (5, 2, 3, 3, 129, 3, 3, 1),       # one pixel per strip
    (1, 36, 7, 70, 72, 3, 3, 1),      # K = 324
]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_seg_waves_edges(shape, dtype, monkeypatch):
    N, Ci, H, W, Co, Kh, Kw, s = shape
    x, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 41)
    xi, wi = workloads.draw(N, Ci, H, W, Co, Kh, Kw, 42, dist="int2")
    ref = torch.from_numpy(oracle.conv(xi.double().numpy(), wi.double().numpy(), s)).to(dtype)
    for v in VARIANTS:
        monkeypatch.setenv("IM2WIN_FP16_SEG", v)
        if v == "w128" and Kh == 11:   # 128 rows of 368 taps and eight 9 KB spans: past 160 KiB
            with pytest.raises(pkg.Im2winError):
                pkg.conv_im2win_kernel_name(*shape, dtype)
            continue
        assert_kernel(shape, dtype, "IM2WIN_FP16_SEG", v)
        say("segment waves", v, shape, dtype)
        r = Run(x, w, s, dtype)
        check_full(r, x, w)
        r.check_workspace_guard()
        r.check_out_guards()
        first = r.out.clone()
        r.rerun_conv()
        assert torch.equal(first.view(torch.int16), r.out.view(torch.int16))
        assert torch.equal(Run(xi, wi, s, dtype).out.cpu(), ref), v


@pytest.mark.parametrize("Ci,s", [(3, 1), (2, 1), (4, 1)])
def test_seg_waves_ignore_next_column(Ci, s, monkeypatch):
    x, w = workloads.draw(1, Ci, 5, 50, 24, 3, 3, 9)
    x[:, :, 40:, :] = float("inf")
    ref = torch.from_numpy(oracle.conv(x[:, :, :40, :].half().double().numpy(), w.half().double().numpy(), s))
    for v in VARIANTS:
        monkeypatch.setenv("IM2WIN_FP16_SEG", v)
        out = Run(x, w, s, torch.float16).out.double().cpu()
        assert torch.isfinite(out[:, :, :38]).all()
        assert (out[:, :, :38] - ref).abs().max() < 0.02
        assert not torch.isfinite(out[:, :, 38:]).any()


def test_seg_waves_refused_where_lds_ends():
    import os
    os.environ["IM2WIN_FP16_SEG"] = "w128"
    try:
        with pytest.raises(pkg.Im2winError):   # 128 rows of 1954 taps
            pkg.conv_im2win_kernel_name(1, 217, 9, 9, 128, 3, 3, 1, "f16")
    finally:
        del os.environ["IM2WIN_FP16_SEG"]


def test_seg_waves_two_threads(monkeypatch):
    """Two host threads, each with its stream and a layer of its own LDS size
    on one kernel instance, in turn: every call launches and gives the bits of
    a single-threaded one."""
    import threading
    monkeypatch.setenv("IM2WIN_FP16_SEG", "w32")
    dt = torch.float16
    jobs = []
    for k, shape in enumerate([(3, 3, 40, 41, 40, 7, 5, 1), (3, 3, 40, 41, 40, 7, 7, 1)]):
        x, w = workloads.draw(*shape[:7], 43 + k)
        assert pkg.conv_im2win_kernel_name(*shape, dt) == "conv_fp16_seg w32"
        jobs.append((shape, Run(x, w, shape[7], dt), torch.cuda.Stream()))
    refs = [r.out.clone() for _, r, _ in jobs]
    errors = []

    def loop(k):
        (N, Ci, H, W, Co, Kh, Kw, s), r, st = jobs[k]
        try:
            for _ in range(200):
                pkg.conv_im2win_fp16(r.ws, r.wd, r.out, N, Ci, H, W, s, stream=st)
            st.synchronize()
        except Exception as e:
            errors.append(e)

    for _, r, _ in jobs:
        r.out.fill_(float("nan"))
    torch.cuda.synchronize()
    ts = [threading.Thread(target=loop, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for (_, r, _), ref in zip(jobs, refs):
        assert torch.equal(r.out.view(torch.int16), ref.view(torch.int16))
