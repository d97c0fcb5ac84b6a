"""The library's host sources on a replaced HIP runtime (host_runtime.cpp): a
Context that needs no GPU and tells what was launched (test code; not collected)."""
import ctypes
import os
import subprocess

import numpy as np

import paper_1907_12343_amd as hrr

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1907_12343_amd", "csrc")
SOURCES = ["hrr_api.cpp", "hrr_launch.cpp", "hrr_build.cpp", "hrr_build_device_host.cpp", "hrr_serve.cpp"]
_P = ctypes.c_void_p


def build(directory):
    """Compile and load the library; `directory` receives it."""
    so = os.path.join(str(directory), "libhrr_host.so")
    cmd = ["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-ffp-contract=off",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), "-pthread",
           os.path.join(HERE, "host_runtime.cpp"), *[os.path.join(CSRC, s) for s in SOURCES], "-o", so]
    subprocess.run(cmd, check=True)
    lib = ctypes.CDLL(so)
    for name, (res, args) in hrr.SIGNATURES.items():
        getattr(lib, name).restype = res
        getattr(lib, name).argtypes = args
    for name in ("host_used", "host_blocks", "host_log"):
        getattr(lib, name).restype = ctypes.c_size_t
    lib.host_spread.argtypes = [ctypes.c_float]
    lib.host_limit.argtypes = [ctypes.c_size_t]
    lib.host_fail_new.argtypes = [ctypes.c_long]
    lib.host_log.argtypes = [_P, ctypes.c_size_t]
    return lib


class HostContext:
    """hrr_ctx on the replaced runtime.  Calls return the hrr_status."""

    def __init__(self, lib):
        self.lib = lib
        tile = np.arange(4096, dtype=np.uint32) << np.uint32(20)
        h = _P()
        assert lib.hrr_create(0, tile.ctypes.data, ctypes.byref(h)) == hrr.HRR_OK
        self.handle = h.value
        self.log()

    def close(self):
        self.lib.hrr_destroy(self.handle)

    def log(self):
        """The lines noted since the last call."""
        buf = ctypes.create_string_buffer(1 << 20)
        assert self.lib.host_log(buf, len(buf)) <= len(buf)
        return buf.value.decode().splitlines()

    def error(self):
        return self.lib.hrr_last_error(self.handle).decode()

    def build(self, n_lights, device=True, leaf=1):
        """(status, handle) of a build of n_lights lights of a fixed sequence."""
        lights = np.ascontiguousarray(np.random.default_rng(5).random((n_lights, 3), dtype=np.float32))
        h = _P()
        if device:
            st = self.lib.hrr_build_hierarchy_device(self.handle, lights.ctypes.data, n_lights, leaf, None, None,
                                                     ctypes.byref(h))
        else:
            st = self.lib.hrr_build_hierarchy(self.handle, lights.ctypes.data, n_lights, leaf, None, ctypes.byref(h))
        return st, h.value

    def hierarchy(self, n_lights, **kw):
        st, h = self.build(n_lights, **kw)
        assert st == hrr.HRR_OK, self.error()
        return h

    def free(self, h):
        self.lib.hrr_free_hierarchy(self.handle, h)

    def eyes(self, n):
        return hrr.HrrEyes(0x1000, n, 64, 0, 0)   # never read

    def traverse(self, h, n_eyes, capacity, s=1e-4, pairs=0x2000, **opt):
        E, o, n = self.eyes(n_eyes), hrr._opts(**opt), ctypes.c_uint64()
        return self.lib.hrr_traverse(self.handle, h, ctypes.byref(E), s, ctypes.byref(o), pairs if capacity else None, None,
                                     capacity, ctypes.byref(n), None, None)

    def noalloc(self, h, n_eyes, capacity, s=1e-4, **opt):
        E, o = self.eyes(n_eyes), hrr._opts(**opt)
        return self.lib.hrr_traverse_noalloc(self.handle, h, ctypes.byref(E), s, ctypes.byref(o), 0x2000 if capacity else None,
                                             None, capacity, 0x3000, None)

    def batched(self, items, pairs=0x2000, **opt):
        """items: (hierarchy, eyes, s, capacity); (status, counts)."""
        arr = (hrr.HrrWorkItem * len(items))()
        at = 0
        for k, (h, n, s, cap) in enumerate(items):
            arr[k] = hrr.HrrWorkItem(h, self.eyes(n), s, 0, at, cap)
            at += cap
        counts = np.zeros(len(items), np.uint64)
        o = hrr._opts(**opt)
        st = self.lib.hrr_traverse_batched(self.handle, arr, len(items), ctypes.byref(o), pairs, None, counts.ctypes.data,
                                           None, None)
        return st, counts
