"""Builds and calls libcrmath_probe.so: the kernels' device math over arrays (crmath_probe.hip)."""
import ctypes as C
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "crmath_probe.hip")
LIB = os.path.join(HERE, "libcrmath_probe.so")
if os.path.dirname(HERE) not in sys.path:
    sys.path.insert(0, os.path.dirname(HERE))

(SIN, COS, SIN_OF_BOTH, COS_OF_BOTH, EXP, LOG, QUOT, ROOT, QUOT_BY_ROOT, FAST_SIN, FAST_COS, DD_SIN,
 DD_COS) = range(13)


def build():
    from paper_1311_5551_amd.build import FLAGS, HIPCC
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.run([HIPCC] + FLAGS + ["-shared", SRC, "-o", tmp], check=True, stderr=subprocess.DEVNULL)
    os.replace(tmp, LIB)


def lib():
    if not os.path.exists(LIB):
        build()
    import torch  # noqa: F401  (its HIP runtime first, as capi.lib does)
    L = C.CDLL(LIB)
    L.probe_f64.argtypes = [C.c_int] + [C.c_void_p] * 4 + [C.c_long]
    L.probe_f32.argtypes = [C.c_int] + [C.c_void_p] * 3 + [C.c_long]
    return L


def call(fn, a, b=None):
    """fn over the numpy arrays a and b (FP64 or FP32); FP64: (results, second words)."""
    import numpy as np
    import torch
    a = np.ascontiguousarray(a)
    d = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (a, a if b is None else b)]
    out = [torch.empty_like(d[0]) for _ in range(2)]
    assert d[0].shape == d[1].shape and d[0].dtype == d[1].dtype
    torch.cuda.synchronize()
    p = [t.data_ptr() for t in d + out]
    e = lib().probe_f64(fn, *p, a.size) if a.dtype == np.float64 else lib().probe_f32(fn, *p[:3], a.size)
    assert e == 0, "HIP error %d" % e
    return tuple(t.cpu().numpy() for t in out) if a.dtype == np.float64 else out[0].cpu().numpy()
