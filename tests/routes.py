"""Which kernels the plans pick for a shape, asked of the planning code (plan_probe.hip), for the host tests of the routes."""
import ctypes
import functools
import os
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=None)
def _probe():
    from paper_2509_14279_amd import build as b
    objects = [os.path.join(b.OBJ, s.replace(".hip", ".o")) for s in b.sources() if s != "fdl_api.hip"]
    if not all(map(os.path.exists, objects)):
        pytest.skip("the library was not built here")
    d = tempfile.mkdtemp(prefix="fdl_routes_")
    obj, lib = os.path.join(d, "probe.o"), os.path.join(d, "probe.so")
    for cmd in ([b.HIPCC, *b.FLAGS, "-O1", "-c", os.path.join(HERE, "plan_probe.hip"), "-o", obj],
                [b.HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, obj, *objects]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
    f = ctypes.CDLL(lib).plan_probe
    f.restype = ctypes.c_char_p
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_int64] * 3
    return f


def route(op, dtype, M, K, N):
    """op: "block", "relu" (both: forward product, gradients, pitch of dZ) or "ffn" (gate and up products, down product)."""
    text = _probe()({"block": 0, "relu": 1, "ffn": 2}[op], {"f32": 0, "bf16": 1}[dtype], M, K, N).decode()
    return text.split(" | ")
