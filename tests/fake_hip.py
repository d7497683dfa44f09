"""Runs Python code against libspkadd.so and the stand-in HIP runtime of fake_hip.cpp, in a
process of its own (without torch, which brings the real runtime)."""
import json
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes, json, sys
sys.path.insert(0, {root!r})
F = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
F.fake_limit.argtypes = [ctypes.c_size_t]
for f in ("fake_used", "fake_peak", "fake_blocks"):
    getattr(F, f).restype = ctypes.c_size_t
F.fake_log.restype = ctypes.c_char_p
from paper_2112_10223_amd import binding as B
L = B.lib()
BINS = (ctypes.c_int * (F.fake_bin_win() + 1)).in_dll(F, "fake_bins")
WINDOWS, TOTAL = ctypes.c_int.in_dll(F, "fake_windows"), ctypes.c_longlong.in_dll(F, "fake_total")
G1, G3, WIN = F.fake_bin_g1(), F.fake_bin_g3(), F.fake_bin_win()
BLOCK = ctypes.create_string_buffer(4096)
ADDR = ctypes.addressof(BLOCK)


def log():
    return [F.fake_log(i).decode().split() for i in range(F.fake_log_size())]


def stream(dev, i=0):
    return ctypes.c_void_p(0x1000 * (dev + 1) + i)


class Sum:
    """One sum through the C calls, whose statuses it keeps; the kernels do not run, so that
    every input array is the same small block."""

    def __init__(self, m, n, k, dtype=0, **opts):
        self.m, self.n, self.k, self.dtype = m, n, k, dtype
        self.o = B.make_opts(**opts)
        self.ptrs = (ctypes.c_void_p * k)(*[ADDR] * k)
        self.h = ctypes.c_void_p()

    def plan(self, s):
        return L.spkadd_plan(ctypes.byref(self.h), self.m, self.n, self.k, self.ptrs, self.ptrs, self.dtype,
                             ctypes.byref(self.o), s)

    def symbolic(self, s):
        self.nnz = ctypes.c_int64()
        return L.spkadd_symbolic(self.h, ADDR, ctypes.byref(self.nnz), s)

    def numeric(self, s):
        return L.spkadd_numeric(self.h, self.ptrs, ADDR, ADDR, s)

    def free(self):
        return L.spkadd_free(self.h)

    def all(self, s):
        st = [self.plan(s)]
        if st[-1] == 0:
            st.append(self.symbolic(s))
        if st[-1] == 0 and len(st) == 2:
            st.append(self.numeric(s))
        self.message = L.spkadd_last_error().decode()
        if self.h:
            self.free()
        return st

    def noalloc(self, s):
        nnz = ctypes.c_int64(-1)
        return L.spkadd_sum_noalloc(self.m, self.n, self.k, self.ptrs, self.ptrs, self.ptrs, self.dtype,
                                    ctypes.byref(self.o), ADDR, ADDR, ADDR, 1 << 30, ctypes.byref(nnz), s)
'''

_built = {}


def build(folder) -> str:
    if "so" not in _built:
        so = os.path.join(str(folder), "libfakehip.so")
        cmd = ["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w", "-I/opt/rocm/include",
               "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2112_10223_amd", "csrc"),
               os.path.join(HERE, "fake_hip.cpp"), "-o", so]
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-4000:]
        _built["so"] = so
    return _built["so"]


def run(folder, code):
    """The value of `out` that the code leaves."""
    text = PRELUDE.format(root=ROOT, fake=build(folder)) + textwrap.dedent(code) + "\nprint('\\n' + json.dumps(out))\n"
    res = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    return json.loads(res.stdout.strip().splitlines()[-1])
