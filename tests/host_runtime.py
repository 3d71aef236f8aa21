"""The library's host code on the stand-in for the HIP runtime in ``tests/hip_stub``: builds it and
wraps what the tests of the host path need."""
import contextlib
import ctypes as C
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_06310_amd", "csrc")
BIG = 1 << 20   # floats of an output buffer


def build(folder, wide=False):
    """wide: with the separable product for graphs of many vertices, which takes pairs from the other forms."""
    so = os.path.join(str(folder), "libmgk_hoststub%s.so" % ("_wide" if wide else ""))
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-shared", "-pthread", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__=1"]
    cmd += ["-DSTUB_WIDE"] if wide else []
    cmd += ["-I/opt/rocm/include", os.path.join(ROOT, "tests", "hip_stub", "hip_stub.cpp"),
            os.path.join(CSRC, "mgk_host.cpp"), os.path.join(CSRC, "mgk_reorder.cpp"), "-o", so]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-4000:]
    return so


class Host:
    """One context on the stand-in.  Streams are small whole numbers."""

    def __init__(self, so, device=0):
        self.lib = C.CDLL(so)
        for name in ("stub_log", "stub_violations", "mgk_last_error"):
            getattr(self.lib, name).restype = C.c_char_p
        for name in ("stub_in_use", "stub_pinned", "mgk_launch_log"):
            getattr(self.lib, name).restype = C.c_int64
        self.lib.stub_reset()
        self.ctx = C.c_void_p()
        assert self.lib.mgk_create(C.byref(self.ctx), device) == 0
        self.K = np.zeros(BIG, np.float32)

    def destroy(self):
        self.lib.mgk_destroy(self.ctx)
        self.ctx = None

    def set(self, name, *args):
        """mgk_set_<name>"""
        assert getattr(self.lib, "mgk_set_" + name)(self.ctx, *[C.c_float(a) if isinstance(a, float) else a for a in args]) == 0

    def load(self, wb, reorder=0):
        p = lambda a, t: np.ascontiguousarray(a, t).ctypes.data_as(C.c_void_p)
        keep = [np.ascontiguousarray(a, t) for a, t in ((wb.vtx_off, np.int64), (wb.vtx_label, np.int32), (wb.edge_off, np.int64),
                                                        (wb.src, np.int32), (wb.dst, np.int32), (wb.weight, np.float32),
                                                        (wb.edge_label, np.float32))]
        vo, vl, eo, s, d, w, e = [a.ctypes.data_as(C.c_void_p) for a in keep]
        h = C.c_void_p()
        st = self.lib.mgk_load_graphs(self.ctx, len(wb.vtx_off) - 1, vo, vl, None, eo, s, d, w, e, reorder, C.byref(h))
        assert st == 0, self.error()
        return h

    def free(self, batch):
        self.lib.mgk_free_batch(self.ctx, batch)

    def error(self):
        return self.lib.mgk_last_error(self.ctx).decode()

    def out(self):
        return self.K.ctypes.data_as(C.c_void_p)

    def gram(self, batch, stream=0):
        return self.lib.mgk_gram(self.ctx, batch, self.out(), None, None, C.c_void_p(stream))

    def pairs(self, X, Y, i, j, stream=0, entry="mgk_pairs"):
        i, j = np.ascontiguousarray(i, np.int32), np.ascontiguousarray(j, np.int32)
        return getattr(self.lib, entry)(self.ctx, X, Y, C.c_int64(len(i)), i.ctypes.data_as(C.c_void_p), j.ctypes.data_as(C.c_void_p),
                                        self.out(), None, None, C.c_void_p(stream))

    def hold(self, stream):
        self.lib.stub_hold(C.c_void_p(stream))

    @contextlib.contextmanager
    def recording(self, stream):
        self.lib.stub_record(C.c_void_p(stream), 1)
        yield
        self.lib.stub_record(C.c_void_p(stream), 0)

    def count(self, what):
        return self.lib.stub_count(what.encode())

    def log(self):
        return self.lib.stub_log().decode()

    def violations(self):
        return self.lib.stub_violations().decode()

    def launch_log(self):
        buf = C.create_string_buffer(1 << 16)
        self.lib.mgk_launch_log(self.ctx, buf, C.c_int64(len(buf)))
        return buf.value.decode()
