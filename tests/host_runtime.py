"""The host library on the recording runtime (tests/c/recording_runtime.cpp): work plans, workspaces,
copies and launches without a GPU.  For a process of its own, in which nothing else has loaded libfmb.so."""
from __future__ import annotations

import atexit
import ctypes
import os
import shutil
import subprocess
import tempfile

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
OK, SHAPE, HIP, OOM = 0, 2, 3, 4
COUNTS = ("allocations", "copies", "overwrites", "refused", "syncs")


class Runtime:
    def __init__(self, root=ROOT):
        tmp = tempfile.mkdtemp(prefix="fmb_rr_")
        atexit.register(shutil.rmtree, tmp, True)
        out = os.path.join(tmp, "rr.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                        "-I" + os.path.join(root, "paper_2308_14737_amd", "csrc"),
                        os.path.join(HERE, "c", "recording_runtime.cpp"), "-o", out], check=True)
        self.rr = ctypes.CDLL(out, mode=ctypes.RTLD_GLOBAL)
        for f in ("rr_count", "rr_in_use"):
            getattr(self.rr, f).restype = ctypes.c_long
        self.rr.rr_name.restype = ctypes.c_char_p
        self.rr.rr_set_limit.argtypes = [ctypes.c_long]
        self.lib = ctypes.CDLL(os.path.join(root, "paper_2308_14737_amd", "libfmb.so"))
        self.lib.fmb_last_error.restype = ctypes.c_char_p

    def count(self, what):
        return self.rr.rr_count(COUNTS.index(what))

    def launches(self):
        """[(kernel, grid, items or None)] since the last call; an item is (view, ray0, span, g0, gc, slots, poff, moff)."""
        res = []
        for i in range(self.rr.rr_launches()):
            grid = (ctypes.c_uint * 3)()
            self.rr.rr_grid(i, grid)
            n = self.rr.rr_items(i, None, 0)
            items = np.zeros((max(n, 1), 8), np.int32)
            self.rr.rr_items(i, items.ctypes.data_as(ctypes.c_void_p), n)
            res.append((self.rr.rr_name(i).decode(), tuple(grid), items[:n]))
        self.rr.rr_clear()
        return res


PTR = ctypes.c_void_p(1 << 20)  # a device address of the caller's (never read)


class Scene:
    """A scene of n Gaussians through the C ABI, its buffers at made-up addresses."""

    def __init__(self, rt: Runtime, n: int, stream: int = 0):
        self.rt, self.n, self.stream = rt, n, ctypes.c_void_p(stream)
        self.h = ctypes.c_void_p()
        self.check(rt.lib.fmb_scene_create(ctypes.byref(self.h), n, PTR, PTR, PTR, PTR, ctypes.c_float(1.0)))

    def check(self, rc, want=OK):
        assert rc == want, (rc, self.rt.lib.fmb_last_error())
        return rc

    def set_cameras(self, hw):
        hw = np.asarray(hw, np.int32)
        self.check(self.rt.lib.fmb_set_cameras(self.h, len(hw), PTR, PTR, hw.ctypes.data_as(ctypes.c_void_p), None, None))

    def set_rays(self, counts):
        c = np.asarray(counts, np.int32)
        self.check(self.rt.lib.fmb_set_rays(self.h, len(c), PTR, PTR, c.ctypes.data_as(ctypes.c_void_p), PTR, None, None))

    def set_model(self, composite):
        self.check(self.rt.lib.fmb_set_model(self.h, None, int(composite)))

    def set_colors(self, on=True):
        self.check(self.rt.lib.fmb_set_colors(self.h, None, PTR if on else None))

    def set_variants(self, fwd, bwd):
        self.check(self.rt.lib.fmb_set_config(self.h, None, fwd, bwd, 1, 1))

    def render(self, normal=False, color=False):
        return self.rt.lib.fmb_render(self.h, PTR, PTR, PTR if normal else None, None, PTR if color else None, PTR, self.stream)

    def backward(self, normal=False, color=False, noalloc=False):
        f = self.rt.lib.fmb_backward_noalloc if noalloc else self.rt.lib.fmb_backward
        return f(self.h, PTR, PTR, PTR if normal else None, None, PTR if color else None, PTR, PTR if color else None, PTR,
                 PTR, PTR, PTR, PTR if color else None, PTR, self.stream)

    def split(self):
        return self.rt.lib.fmb_split_statistic(self.h, None, PTR, PTR, PTR, self.stream)

    def autotune(self):
        return self.rt.lib.fmb_autotune(self.h, None, PTR, PTR, None, None, None, PTR, PTR, PTR, None, None, None,
                                        PTR, PTR, PTR, None, PTR, None, self.stream)
