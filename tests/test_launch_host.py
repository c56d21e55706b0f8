"""What the conv calls ask of the HIP runtime, on the host: the library is
loaded behind stand-ins that record launches and function attributes
(hip_calls.cpp), in a process of its own.  No call here reaches a GPU."""
import ctypes
import os
import subprocess
import sys
import textwrap

import pytest

import paper_2608_20725_amd as pkg

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PRELUDE = '''
import ctypes, os, sys
i64 = ctypes.c_int64
class Call(ctypes.Structure):
    _fields_ = [(n, ctypes.c_longlong) for n in ("kind", "func", "value", "gx", "gy", "block")]
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
lib.conv_workspace_bytes.restype = i64
lib.conv_workspace_bytes.argtypes = [i64] * 8 + [ctypes.c_int]
fns = {0: lib.conv_im2win_fp32, 1: lib.conv_im2win_fp16, 2: lib.conv_im2win_bf16}
for f in fns.values():
    f.argtypes = [ctypes.c_void_p, i64, ctypes.c_void_p, ctypes.c_void_p] + [i64] * 8 + [ctypes.c_void_p]
lib.conv_im2win_transform.argtypes = [ctypes.c_void_p, ctypes.c_void_p] + [i64] * 9 + [ctypes.c_int, ctypes.c_void_p]
ATTR, LAUNCH, QUERY = 0, 1, 2
def transform(shape, dt, kernel=None):
    """The launch of a layer's transform, the kernel forced or the default."""
    os.environ["IM2WIN_TRANSFORM_KERNEL"] = kernel or ""
    need = lib.conv_workspace_bytes(*shape, dt)
    N, Ci, H, W, Co, Kh, Kw, s = shape
    rc = lib.conv_im2win_transform(1 << 40, 1 << 44, need, N, Ci, H, W, Co, Kh, Kw, s, dt, None)
    assert rc == 0, rc
    (c,) = calls()
    return c
def conv(shape, dt):
    """The conv call of a layer (buffers that no call touches)."""
    need = lib.conv_workspace_bytes(*shape, dt)
    assert need > 0, need
    N, Ci, H, W, Co, Kh, Kw, s = shape
    rc = fns[dt](1 << 40, need, 1 << 44, 1 << 48, N, Ci, H, W, Co, Kh, Kw, s, None)
    assert rc == 0, rc
def calls():
    a = (Call * 65536)()
    return list(a[:shim.shim_calls(a, 65536)])
'''


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    if not os.path.exists(pkg.library_path()):
        from paper_2608_20725_amd import build
        build.build()
    out = str(tmp_path_factory.mktemp("shim") / "hip_calls.so")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_calls.cpp"), "-o", out],
                   check=True, capture_output=True)
    return out


def run(shim, body):
    env = {k: v for k, v in os.environ.items() if not k.startswith("IM2WIN_")}
    p = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), shim, pkg.library_path()],
                       capture_output=True, text=True, env=env, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr


def test_segment_kernel_lds_limit_is_the_same_for_every_layer(shim):
    """Two layers that run one instance of the one-wave segment kernel with
    different LDS sizes: the function's limit does not depend on which layer
    set it last, and covers every launch."""
    run(shim, '''
    small, large = (64, 3, 60, 60, 96, 7, 5, 1), (64, 3, 60, 60, 96, 7, 7, 1)
    seen = {}
    for dt in (1, 2):
        for shape in (large, small, large):
            conv(shape, dt)
            for c in calls():
                seen.setdefault(c.func, []).append(c)
    both = [v for f, v in seen.items() if len({c.value for c in v if c.kind == LAUNCH and c.value}) == 2]
    assert len(both) == 2, "the layers no longer share an instance"
    for v in both:
        limits = {c.value for c in v if c.kind == ATTR}
        assert len(limits) == 1, limits
        assert max(c.value for c in v if c.kind == LAUNCH) <= limits.pop() <= 160 * 1024
    ''')


def test_segment_kernel_repeated_call_asks_the_driver_nothing(shim):
    """A second call of the same layer, from any thread, is one launch with
    the grid of the first."""
    run(shim, '''
    import threading
    shape = (64, 3, 60, 60, 96, 7, 7, 1)
    conv(shape, 1)
    first = calls()
    assert [c.kind for c in first if c.kind != LAUNCH] and first[-1].kind == LAUNCH
    ts = [threading.Thread(target=conv, args=(shape, 1)) for _ in range(4)]
    for t in ts: t.start()
    for t in ts: t.join()
    again = calls()
    assert len(again) == 4 and all(c.kind == LAUNCH for c in again), [c.kind for c in again]
    for c in again:
        assert (c.func, c.value, c.gx, c.gy, c.block) == tuple(getattr(first[-1], n) for n in
                                                               ("func", "value", "gx", "gy", "block"))
    ''')


@pytest.mark.parametrize("shape,dt,want", [
    # narrow images: a piece of many strips is many short rows for four waves
    ((125, 3, 90, 13, 16, 7, 7, 2), 1, "gather"), ((73, 3, 68, 9, 16, 5, 5, 1), 2, "gather"),
    ((67, 3, 57, 14, 16, 7, 7, 1), 2, "gather"), ((108, 3, 35, 35, 16, 5, 5, 1), 1, "gather"),
    ((113, 3, 98, 15, 16, 7, 7, 2), 0, "3ch"), ((112, 3, 108, 39, 16, 3, 3, 2), 0, "3ch"),
    # small 3-channel tensors: one load per pixel
    ((1, 3, 32, 32, 16, 3, 3, 1), 0, "3ch"), ((112, 3, 27, 27, 16, 3, 3, 1), 1, "3ch"),
    # long runs of 2-byte units
    ((1, 299, 65, 65, 16, 1, 1, 1), 1, "gather"), ((16, 209, 10, 10, 16, 5, 5, 1), 1, "gather"),
    # where pieces are ahead: the stems, inner layers off 8 channels, small ones of one row pass
    ((128, 3, 227, 227, 96, 11, 11, 4), 1, "pieces"), ((32, 3, 230, 230, 64, 7, 7, 2), 0, "pieces"),
    ((128, 3, 224, 224, 64, 3, 3, 1), 1, "pieces"), ((128, 3, 224, 224, 64, 3, 3, 1), 0, "pieces"),
    ((92, 52, 81, 81, 51, 3, 3, 1), 1, "pieces"), ((7, 36, 31, 45, 100, 3, 5, 2), 1, "pieces"),
    ((128, 100, 28, 28, 100, 1, 1, 1), 1, "pieces"),
])
def test_transform_kernel_by_its_row_passes(shim, shape, dt, want):
    """The default transform of unaligned channel counts: the element gather,
    the one-load-per-pixel gather of 3 channels, or pieces put together in LDS."""
    run(shim, '''
    shape, dt, want = %r, %r, %r
    got = transform(shape, dt).func
    forced = {k: transform(shape, dt, k).func for k in ("pieces", "gather")}
    kind = next((k for k, f in forced.items() if f == got), "3ch")
    assert kind == want, kind
    ''' % (shape, dt, want))


def test_transform_pieces_grid(shim):
    """Strips share a piece only beyond four pieces per CU."""
    run(shim, '''
    for shape, dt in (((110, 3, 110, 15, 16, 3, 3, 1), 1), ((300, 5, 40, 9, 16, 3, 3, 1), 0)):
        assert transform(shape, dt, "pieces").gx >= 1024
    ''')
