"""The path captured in a HIP graph (torch.cuda.graph over the C-ABI calls,
which launch on the current stream): every replay must reproduce the eager
result bit for bit, with eager work, input changes and synchronisations
between the replays (the library records no memset nodes: the transform
zeroes its pad with a kernel)."""
import pytest
import torch

import paper_2608_20725_amd as pkg
from gpu_util import say
from paper_2608_20725_amd import workloads

pytestmark = pytest.mark.gpu

CASES = [
    ((4, 64, 20, 20, 64, 3, 3, 1), torch.float32),
    ((4, 64, 20, 20, 64, 3, 3, 1), torch.float16),
    ((2, 3, 31, 29, 40, 5, 5, 2), torch.float32),   # unaligned windows: the element gather
    ((2, 3, 31, 29, 40, 5, 5, 2), torch.bfloat16),
    ((2, 256, 9, 9, 300, 3, 3, 1), torch.float16),   # several channel tiles, XCD-aware order
    # one layer per family: (shape, dtype, kernel, the variable that forces it)
    ((2, 64, 20, 20, 64, 3, 3, 1), torch.float16, "conv_fp16_pipe c64p64s4", "IM2WIN_FP16_TILE"),
    ((2, 64, 20, 20, 130, 3, 3, 1), torch.bfloat16, "conv_fp16_pipe c128p128s1", "IM2WIN_FP16_TILE"),
    ((64, 64, 58, 58, 64, 3, 3, 1), torch.float16, "conv_fp16_col k3c64p128t32s2", None),   # persistent launch
    ((4, 8, 20, 20, 40, 3, 3, 1), torch.bfloat16, "conv_fp16_col k3c64p128t32s2", "IM2WIN_FP16_COL"),
    ((3, 272, 37, 36, 360, 7, 7, 1), torch.float16, "conv_fp16_pipe c128p128s2 k4", None),  # two conv kernels
    ((12, 3, 60, 61, 96, 7, 7, 2), torch.float16, "conv_fp16_seg w32", "IM2WIN_FP16_SEG"),
    ((12, 3, 60, 61, 96, 7, 7, 2), torch.bfloat16, "conv_fp16_seg w96", "IM2WIN_FP16_SEG"),
    ((2, 3, 60, 61, 64, 7, 7, 2), torch.float16, "conv_fp16_seg s64p128g1024", "IM2WIN_FP16_SEG"),
    ((2, 3, 60, 61, 64, 3, 3, 1), torch.float16, "conv_fp16_stem m2k2", None),
    ((1, 3, 32, 32, 16, 3, 3, 1), torch.float32, "conv_fp32_stem k27c8", None),
    ((2, 3, 60, 61, 64, 3, 3, 1), torch.float32, "conv_fp32_stem k27", "IM2WIN_FP32_KERNEL=stem"),
    ((1, 256, 16, 16, 256, 3, 3, 1), torch.float32, "conv_fp32_dma p4c4l8s2k16t8w8", None),
]


def _eager(x, w, s, dtype):
    N, H, W, Ci = x.shape
    Kh, Kw, _, Co = w.shape
    Ho, Wo = pkg.conv_output_dims(H, W, Kh, Kw, s)
    ws = torch.empty(pkg.conv_workspace_bytes(N, Ci, H, W, Co, Kh, Kw, s, dtype), dtype=torch.uint8, device="cuda")
    out = torch.empty((N, Ho, Wo, Co), dtype=dtype, device="cuda")
    pkg.conv_im2win_transform(x, ws, Co, Kh, Kw, s)
    pkg.conv_for_dtype(dtype)(ws, w, out, N, Ci, H, W, s)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + "-" + str(c[1])[6:] + "".join("-" + k.replace(" ", "-") for k in c[2:3]))
def test_graph_replays_match_eager(case, monkeypatch):
    (N, Ci, H, W, Co, Kh, Kw, s), dtype = case[:2]
    say("graph", case)
    if len(case) > 2:
        kernel, var = case[2:]
        if var:
            k, _, v = var.partition("=")
            monkeypatch.setenv(k, v or kernel.split()[1])
        assert pkg.conv_im2win_kernel_name(N, Ci, H, W, Co, Kh, Kw, s, dtype) == kernel
    xa, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, seed=61)
    xb, _ = workloads.draw(N, Ci, H, W, Co, Kh, Kw, seed=62)
    xa, xb, w = xa.to(dtype).cuda(), xb.to(dtype).cuda(), w.to(dtype).cuda()
    ref_a, ref_b = _eager(xa, w, s, dtype), _eager(xb, w, s, dtype)
    bits = torch.int32 if dtype == torch.float32 else torch.int16
    assert not torch.equal(ref_a.view(bits), ref_b.view(bits))

    x = xa.clone()
    Ho, Wo = pkg.conv_output_dims(H, W, Kh, Kw, s)
    ws = torch.empty(pkg.conv_workspace_bytes(N, Ci, H, W, Co, Kh, Kw, s, dtype), dtype=torch.uint8, device="cuda")
    out = torch.empty((N, Ho, Wo, Co), dtype=dtype, device="cuda")
    conv = pkg.conv_for_dtype(dtype)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):   # one eager call on the capture stream first
        pkg.conv_im2win_transform(x, ws, Co, Kh, Kw, s)
        conv(ws, w, out, N, Ci, H, W, s)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        pkg.conv_im2win_transform(x, ws, Co, Kh, Kw, s)
        conv(ws, w, out, N, Ci, H, W, s)
    torch.cuda.synchronize()
    for rep, (src, ref) in enumerate([(xa, ref_a), (xa, ref_a), (xb, ref_b), (xa, ref_a)]):
        x.copy_(src)
        out.fill_(float("nan"))        # eager work between the replays
        ws[: ws.numel() // 2].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(bits), ref.view(bits)), "replay %d" % rep


def test_capture_after_a_layer_of_the_same_kernel(monkeypatch):
    """The one-wave segment kernel asks the driver for its occupancy when the
    layer before it on the same instance had another LDS size: also inside a
    capture."""
    monkeypatch.setenv("IM2WIN_FP16_SEG", "w32")
    dt = torch.float16
    layers = []
    for k, shape in enumerate([(3, 3, 40, 41, 40, 7, 5, 1), (3, 3, 40, 41, 40, 7, 7, 1)]):
        N, Ci, H, W, Co, Kh, Kw, s = shape
        x, w = workloads.draw(N, Ci, H, W, Co, Kh, Kw, seed=65 + k)
        x, w = x.to(dt).cuda(), w.to(dt).cuda()
        layers.append((shape, x, w, _eager(x, w, s, dt)))   # ends with the second layer's size kept
    (N, Ci, H, W, Co, Kh, Kw, s), x, w, ref = layers[0]
    ws = torch.empty(pkg.conv_workspace_bytes(N, Ci, H, W, Co, Kh, Kw, s, dt), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        pkg.conv_im2win_transform(x, ws, Co, Kh, Kw, s)
        pkg.conv_im2win_fp16(ws, w, out, N, Ci, H, W, s)
    for _ in range(3):
        out.fill_(float("nan"))
        _eager(layers[1][1], layers[1][2], s, dt)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
