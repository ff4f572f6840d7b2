"""The library's host code on a machine without a GPU: gwfa_host.cpp compiled
by g++ with a stand-in for the HIP runtime and the kernels (fake_hip.cpp)."""
import ctypes
import os
import subprocess

import numpy as np

from paper_2206_13574_amd import build, gwfa

_HERE = os.path.dirname(os.path.abspath(__file__))
_P = ctypes.c_void_p
GIB = 1 << 30


def compile_host(out_dir: str) -> str:
    out = os.path.join(out_dir, "libhost.so")
    host = [s for s in build.sources() if s.endswith("gwfa_host.cpp")][0]
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
                        "-Wl,-Bsymbolic", "-I/opt/rocm/include", "-I", os.path.join(os.path.dirname(build._PKG), "include"),
                        "-I", os.path.dirname(host), "-o", out, host, os.path.join(_HERE, "fake_hip.cpp")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


class Host:
    """The entry points and the stand-in's controls of one compiled copy."""

    def __init__(self, path):
        self.lib = ctypes.CDLL(path)
        for name, (res, args) in gwfa._SIGS.items():
            f = getattr(self.lib, name, None)
            if f is not None:
                f.restype, f.argtypes = res, args
        for name in ("fake_used", "fake_cigar_groups", "fake_screen_blocks", "fake_queue_place"):
            getattr(self.lib, name).restype = ctypes.c_int64
        self.lib.fake_memory.argtypes = [ctypes.c_int64]
        self.lib.fake_largest.argtypes = self.lib.fake_new_limit.argtypes = [ctypes.c_int64]

    def reset(self):
        """A device of 288 GiB, nothing failing."""
        self.lib.fake_memory(288 * GIB)
        self.lib.fake_largest(-1)
        self.lib.fake_new_limit(-1)
        for d in range(32):
            self.lib.fake_overflow(d, 0)
        self.lib.fake_clear()

    def context(self, lanes=256, groups=0, dir_log2_max=16, list_cap=1 << 15, dir_factor=16):
        h = _P()
        assert self.lib.gwfa_ctx_create(0, None, ctypes.byref(h)) == 0
        assert self.lib.gwfa_ctx_config(h, lanes, groups, dir_log2_max, list_cap, dir_factor) == 0
        self.lib.gwfa_mlp_load(h, np.zeros(gwfa.MLP_N, np.uint16).ctypes.data_as(_P), gwfa.MLP_N,
                               np.ones(8, np.float32).ctypes.data_as(_P))
        return h

    def graph(self, ctx, n_vtx=4, bases=30):
        off = np.arange(n_vtx + 1, dtype=np.int64) * bases
        h, z = _P(), np.zeros(1, np.int32)
        rc = self.lib.gwfa_graph_create(ctx, n_vtx, np.full(n_vtx * bases, 65, np.uint8).ctypes.data_as(_P),
                                        off.ctypes.data_as(_P), 0, z.ctypes.data_as(_P), z.ctypes.data_as(_P),
                                        ctypes.byref(h))
        return h if rc == 0 else rc

    _buf = np.zeros(1 << 16, np.int64)      # every device argument: read and written by nobody

    def align(self, ctx, graph, n=1000, **kw):
        b = self._buf.ctypes.data_as(_P)
        return self.lib.gwfa_align_batch_dev(ctx, graph, n, b, b, b, None, ctypes.byref(gwfa.opts(**kw)), b, b, 0, b, None)

    def plan(self, ctx, graph, n=1000, **kw):
        b, p = self._buf.ctypes.data_as(_P), _P()
        rc = self.lib.gwfa_plan_create(ctx, graph, n, b, b, b, None, ctypes.byref(gwfa.opts(**kw)), b, b, 0, b,
                                       ctypes.byref(p))
        return rc, p

    def launches(self):
        """(directory size, lanes, groups, queries, records' tier, arenas allocated, bytes a query) of each launch."""
        out = []
        for i in range(self.lib.fake_launches()):
            v = (ctypes.c_int64 * 7)()
            self.lib.fake_launch(i, v)
            out.append(tuple(v))
        self.lib.fake_clear()
        return out

    def dirs(self):
        ls = self.launches()
        assert all(x[5] for x in ls), ls          # no launch on arenas given back
        return [x[0] for x in ls]
