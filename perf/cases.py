"""The calls whose speed counts: convolutions as programs make them through the public entry points.

A case is one layer applied to one batch: transform, filter pack and windowed convolution from an NHWC input
resident on the GPU, with the workspace and the output buffer that a program keeps between calls.  Sizes are
the repository's layer configurations (``workloads.py``) at batches from one image to 128, with the options
its entry points have (zero padding, dilation, mini-batches on two streams, fp32 on the matrix cores).

Fields: ``op`` names the entry points (``conv2d``: im2win_conv2d; ``padded``: conv_im2win_transform_padded and
the precision's conv; ``dilated``: conv_im2win_transform_dilated and conv_im2win_dilated; ``chunked``:
conv_im2win_chunked with a second stream; ``mfma32``: conv_im2win_transform and conv_im2win_fp32_mfma), ``dt``
the element type, and N, Ci, H, W, Co, Kh, Kw, s, pad, dil, chunk the layer (``chunk``: images per mini-batch).
"""
import math

import torch

import paper_2608_20725_amd as im2win

_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _case(name, op, dt, N, Ci, H, W, Co, Kh, Kw, s, pad=0, dil=1, chunk=0):
    return {"name": name, "op": op, "dt": dt, "N": N, "Ci": Ci, "H": H, "W": W, "Co": Co, "Kh": Kh, "Kw": Kw,
            "s": s, "pad": pad, "dil": dil, "chunk": chunk}


def listed():
    return [
        # the smallest call: one small colour image, latency and launches only
        _case("tiny_c3_32_f32", "conv2d", "f32", 1, 3, 32, 32, 16, 3, 3, 1),
        # single-image inference, a middle layer of a residual network with 'same' padding
        _case("image1_c256_14_f16", "padded", "f16", 1, 256, 14, 14, 256, 3, 3, 1, pad=1),
        # a small serving batch in the last stage: long windows over few pixels
        _case("image8_c512_7_bf16", "padded", "bf16", 8, 512, 7, 7, 512, 3, 3, 1, pad=1),
        # odd sizes throughout: channels, extents, a filter that is not square, windows not 16-byte aligned
        _case("ragged_c36_31x45_f16", "conv2d", "f16", 7, 36, 31, 45, 100, 3, 5, 2),
        # atrous layer of a segmentation network
        _case("atrous_c256_28_d2_f16", "dilated", "f16", 32, 256, 28, 28, 256, 3, 3, 1, pad=2, dil=2),
        # large-kernel stem at the training / offline batch
        _case("stem_c3_227_11x11_s4_f16", "conv2d", "f16", 128, 3, 227, 227, 96, 11, 11, 4),
        # 7x7 stem with padding at a mid-size batch, fp32
        _case("stem_c3_224_7x7_s2_f32", "padded", "f32", 32, 3, 224, 224, 64, 7, 7, 2, pad=3),
        # the ordinary 3x3 layer at full batch, fp32 on the vector ALUs
        _case("c64_56_3x3_f32", "conv2d", "f32", 128, 64, 56, 56, 64, 3, 3, 1),
        # the same layer in fp16 with the memory bounded: mini-batches alternating on two streams
        _case("c64_56_3x3_chunks_f16", "chunked", "f16", 128, 64, 56, 56, 64, 3, 3, 1, chunk=32),
        # pointwise layer: a plain matrix product
        _case("c1024_14_1x1_f16", "conv2d", "f16", 128, 1024, 14, 14, 1024, 1, 1, 1),
        # high-resolution 3x3 layer at full batch, bf16
        _case("c64_112_3x3_bf16", "conv2d", "bf16", 128, 64, 112, 112, 128, 3, 3, 1),
        # the largest: 7x7 stride 2 over 64 channels, fp32 on the matrix cores
        _case("c64_224_7x7_s2_mfma_f32", "mfma32", "f32", 128, 64, 224, 224, 64, 7, 7, 2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A layer of the same ranges: stem or inner layer, any batch, type and option; at most 100 GFLOP."""
    while True:
        op = rng.choice(["conv2d", "conv2d", "conv2d", "padded", "padded", "dilated", "chunked", "mfma32"])
        dt = "f32" if op == "mfma32" else rng.choice(["f32", "f16", "bf16"])
        N = _log_int(rng, 1, 128)
        if op in ("conv2d", "padded", "chunked") and rng.random() < 0.25:   # stem
            Ci, H = 3, rng.randint(32, 227)
            K, s = rng.choice([(3, 1), (3, 2), (5, 2), (7, 2), (11, 4)])
            Co = 8 * rng.randint(2, 16)
        else:
            H = _log_int(rng, 7, 112)
            # channels shrink as the extent grows, as in the networks; one in four not a multiple of 8
            Ci = _log_int(rng, 16, max(24, min(1024, 7168 // H)))
            Co = _log_int(rng, 16, max(24, min(1024, 14336 // H)))
            if rng.random() < 0.75:
                Ci, Co = 8 * max(2, Ci // 8), 8 * max(2, Co // 8)
            K, s = rng.choice([(1, 1), (3, 1), (3, 1), (3, 1), (3, 2), (5, 1), (7, 2)])
        W = H if rng.random() < 0.7 else max(7, H + rng.randint(-H // 4, H // 4))
        Kw = K if K == 1 or rng.random() < 0.85 else rng.choice([1, 3, 5])
        dil = rng.choice([1, 2, 3]) if op == "dilated" and K > 1 else 1
        pad = dil * (K - 1) // 2 if op in ("padded", "dilated") else 0
        c = _case("", op, dt, N, Ci, H, W, Co, K, Kw, s, pad=pad, dil=dil,
                  chunk=max(1, -(-N // 4)) if op == "chunked" else 0)
        del c["name"]
        if min(H, W) + 2 * pad < dil * (max(K, Kw) - 1) + 1:
            continue
        if 1e6 <= work(c)["flops"] <= 1e11:
            return c


def _dims(c):
    Hp, Wp = c["H"] + 2 * c["pad"], c["W"] + 2 * c["pad"]
    Ho = (Hp - c["dil"] * (c["Kh"] - 1) - 1) // c["s"] + 1
    Wo = (Wp - c["dil"] * (c["Kw"] - 1) - 1) // c["s"] + 1
    return Hp, Wp, Ho, Wo


def _inputs(c, seed):
    # unit activations and a filter scaled by its fan-in, as after initialisation
    g = torch.Generator("cuda").manual_seed(int(seed))
    k = c["Kh"] * c["Kw"] * c["Ci"]
    x = torch.randn((c["N"], c["H"], c["W"], c["Ci"]), generator=g, device="cuda")
    w = torch.randn((c["Kh"], c["Kw"], c["Ci"], c["Co"]), generator=g, device="cuda") * math.sqrt(2.0 / k)
    return x.to(_DT[c["dt"]]), w.to(_DT[c["dt"]])


def prepare(case, seed):
    c = case
    x, w = _inputs(c, seed)
    Hp, Wp, Ho, Wo = _dims(c)
    layer = (c["N"], c["Ci"], Hp, Wp, c["Co"], c["Kh"], c["Kw"], c["s"])
    st = {"case": c, "x": x, "w": w}
    if c["op"] == "chunked":
        need = im2win.conv_chunked_workspace_bytes(*layer, c["chunk"], True, x.dtype)
        st["aux"] = torch.cuda.Stream()
    elif c["op"] == "dilated":
        need = im2win.conv_workspace_bytes_dilated(*layer, c["dil"], x.dtype)
    else:
        need = im2win.conv_workspace_bytes(*layer, x.dtype)
    st["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    st["out"] = torch.empty((c["N"], Ho, Wo, c["Co"]), dtype=x.dtype, device="cuda")
    return st


def run(state):
    c, x, w, ws, out = (state[k] for k in ("case", "x", "w", "ws", "out"))
    op, s = c["op"], c["s"]
    if op == "conv2d":
        im2win.im2win_conv2d(x, w, s, ws=ws, out=out)
    elif op == "chunked":
        im2win.conv_im2win_chunked(x, w, out, ws, s, c["chunk"], aux_stream=state["aux"])
    else:
        N, Ci, Co, Kh, Kw, pad = c["N"], c["Ci"], c["Co"], c["Kh"], c["Kw"], c["pad"]
        Hp, Wp = c["H"] + 2 * pad, c["W"] + 2 * pad
        if op == "padded":
            im2win.conv_im2win_transform_padded(x, ws, Co, Kh, Kw, s, pad, pad)
            im2win.conv_for_dtype(x.dtype)(ws, w, out, N, Ci, Hp, Wp, s)
        elif op == "dilated":
            im2win.conv_im2win_transform_dilated(x, ws, Co, Kh, Kw, s, pad, pad, c["dil"])
            im2win.conv_im2win_dilated(ws, w, out, N, Ci, Hp, Wp, s, c["dil"])
        else:
            im2win.conv_im2win_transform(x, ws, Co, Kh, Kw, s)
            im2win.conv_im2win_fp32_mfma(ws, w, out, N, Ci, Hp, Wp, s)
    return out


def work(case):
    c = case
    _, _, Ho, Wo = _dims(c)
    elt = 4 if c["dt"] == "f32" else 2
    k, pixels = c["Kh"] * c["Kw"] * c["Ci"], c["N"] * Ho * Wo
    return {"bytes": elt * (c["N"] * c["H"] * c["W"] * c["Ci"] + k * c["Co"] + pixels * c["Co"]),
            "flops": 2 * pixels * c["Co"] * k}


def tolerance(case):
    # about four times the distance from the 64-bit result: the rounding of the output in 16 bits, the order
    # of up to 5000 fp32 additions in fp32
    return {"rel": {"f32": 4e-6, "f16": 9e-4, "bf16": 7e-3}[case["dt"]]}


def exact(case, seed):
    c = case
    x, w = _inputs(c, seed)
    _, _, Ho, Wo = _dims(c)
    p, d, s = c["pad"], c["dil"], c["s"]
    xp = torch.nn.functional.pad(x, (0, 0, p, p, p, p)).double()
    wd = w.double()
    out = torch.zeros((c["N"] * Ho * Wo, c["Co"]), dtype=torch.float64, device="cuda")
    for u in range(c["Kh"]):
        for v in range(c["Kw"]):
            rows = xp[:, u * d:u * d + (Ho - 1) * s + 1:s, v * d:v * d + (Wo - 1) * s + 1:s, :]
            out.addmm_(rows.reshape(-1, c["Ci"]), wd[u, v])
    return out.view(c["N"], Ho, Wo, c["Co"])
