"""Runs the library's host code on the CPU in a process of its own, on the
stand-in runtime of hip_standin.cpp (kernels are recorded, not run: the CG
state stays zero, so a solve ends after its first chunk of steps)."""

import ctypes
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def run(tmp_path, body):
    """Run `body` with `s` (an instance of Host) in scope; its output."""
    so = os.path.join(str(tmp_path), "libstandin.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_standin.cpp")],
                   check=True)
    code = "import sys\nsys.path[:0] = %r\nfrom standin import Host\ns = Host(%r)\n" % ([ROOT, HERE], so)
    r = subprocess.run([sys.executable, "-c", code + textwrap.dedent(body)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


class Host:
    def __init__(self, so):
        import types
        self.hip = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.hip.standin_stream.restype = ctypes.c_void_p
        self.hip.standin_launch.restype = ctypes.c_char_p
        sys.modules.setdefault("torch", types.ModuleType("torch"))  # (the binding loads it only for its runtime)
        import paper_1211_0126_amd as tq
        if not os.path.exists(tq.LIB_PATH):
            from paper_1211_0126_amd.build import build
            build()
        self.tq, self.b = tq, tq.binding
        self.lib = tq.load_library()

    def context(self, dims, nbytes, device=0):
        """A context with its own workspace on a stream of `device`, links
        loaded, launches eager."""
        import numpy as np
        h = ctypes.c_void_p()
        lat = self.b._lattice(dims, 0.1632, 0.004, -1)
        self.hip.hipSetDevice(device)
        assert self.lib.tm_create(ctypes.byref(lat), None, int(nbytes), ctypes.c_void_p(self.hip.standin_stream(device)),
                                  ctypes.byref(h)) == 0, self.lib.tm_last_error(None)
        ctx = self.b.Context.__new__(self.b.Context)
        ctx.lib, ctx.h, ctx.dims, ctx.V, ctx.workspace = self.lib, h, tuple(dims), int(np.prod(dims)), None
        ctx.kappa, ctx.mu, ctx.t_bc, ctx.stream = 0.1632, 0.004, -1, None
        self.tq.tm_gauge_load(ctx, np.zeros((ctx.V, 4, 3, 3), dtype=np.complex128))
        self.tq.tm_set_graphs(ctx, False)
        self.launches()
        return ctx

    def launches(self):
        """[(kernel, (x, y, z))] since the last call."""
        out = []
        for i in range(self.hip.standin_launches()):
            name, *grid = self.hip.standin_launch(i).decode().rsplit(" ", 3)
            out.append((name, tuple(int(v) for v in grid)))
        self.hip.standin_clear()
        return out
