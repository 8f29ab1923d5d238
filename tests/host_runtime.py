"""Runs the library's host side without a GPU, on the runtime of host_runtime.cpp, in a process of its own."""
import ctypes as C
import os
import subprocess
import sys
import types

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build(folder):
    so = os.path.join(str(folder), "host_runtime.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1804_10727_amd", "csrc"), "-o", so,
                    os.path.join(ROOT, "tests", "host_runtime.cpp")], check=True)
    return so


def run(so, script, function, *args):
    """Calls function(runtime, *args) of the script in a process whose HIP runtime is the stand-in."""
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]\n"
            f"import host_runtime; rt = host_runtime.start({so!r})\n"
            f"import {script}; {script}.{function}(rt, *{args!r})\nprint('done')")
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.endswith("done\n"), p.stdout + p.stderr


def start(so):
    rt = C.CDLL(so, mode=C.RTLD_GLOBAL)         # in front of the real runtime for whatever is loaded from here on
    rt.host_error.restype = C.c_char_p
    rt.host_launches.restype = rt.host_max_lds.restype = C.c_long
    rt.host_launches.argtypes = [C.c_char_p]
    rt.host_fail_in.argtypes = [C.c_long]
    rt.host_record.argtypes = [C.c_ulonglong]
    sys.modules["torch"] = types.ModuleType("torch")      # (the binding loads it for its runtime; not wanted here)
    return rt


class Streams:
    """Open streams of a net whose workspace and buffers are addresses only."""

    def __init__(self, net, n, max_seg=1, out_cap=0, workspace_bytes=None, static=False):
        from paper_1804_10727_amd import binding
        self.L, self.check, self.n = binding.load_library(), binding._check, n
        h = C.c_void_p()
        if static:
            self.check(self.L.idf_open_streams_static(net._h, n, max_seg, out_cap, None, C.byref(h)))
        else:
            size = net.query_sizes(n, max_seg, out_cap).workspace_bytes if workspace_bytes is None else workspace_bytes
            self.check(self.L.idf_open_streams(net._h, n, max_seg, out_cap, C.c_void_p(1 << 40), size, None, C.byref(h)))
        self.h = h

    def push(self, n_rows, ids=None):
        import numpy as np
        a = None if ids is None else np.ascontiguousarray(ids, dtype=np.int32)
        self.check(self.L.idf_push_segment(self.h, None if a is None else a.ctypes.data, self.n if a is None else len(a),
                                           C.c_void_p(1 << 50), n_rows))

    def push_pixels(self, x0, n, ids):
        import numpy as np
        a = np.ascontiguousarray(ids, dtype=np.int32)
        self.check(self.L.idf_push_pixels(self.h, a.ctypes.data, len(a), C.c_void_p(1 << 50), x0, n))

    def stats(self, i):
        self.check(self.L.idf_get_stats(self.h, i, None, None, None))

    def read(self, max_rows):
        import numpy as np
        first, cnt = np.zeros(self.n, np.int64), np.zeros(self.n, np.int32)
        self.check(self.L.idf_read_outputs(self.h, None, self.n, C.c_void_p(1 << 51), max_rows, first.ctypes.data, cnt.ctypes.data))
        return cnt

    def close(self):
        self.check(self.L.idf_close_streams(self.h))
