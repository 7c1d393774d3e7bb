"""libchefsi.so's host code without a GPU: the library loaded behind hip_host_stub.cpp.  For a process
of its own (``python -m tests._host <function> ...``), as the stub takes the place of HIP."""
import ctypes as C
import os
import shutil
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))


def build_stub(folder):
    gxx = shutil.which("g++")
    assert gxx, "no host compiler"
    lib = os.path.join(str(folder), "hip_host_stub.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_host_stub.cpp"), "-o", lib],
                   check=True)
    return lib


def run(stub, module, *args):
    """Runs module's main in a process where the stub stands for HIP; its output."""
    r = subprocess.run([sys.executable, "-m", module, stub, *map(str, args)], capture_output=True, text=True,
                       cwd=os.path.dirname(HERE), timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-4000:]
    return r.stdout


class Host:
    """A handle whose device memory is host memory."""

    def __init__(self, stub, prob, precision, max_ns):
        self.stub = C.CDLL(stub, mode=C.RTLD_GLOBAL)
        self.stub.stub_launches.restype = C.c_char_p
        self.stub.stub_null_tables.restype = C.c_long
        self.stub.stub_fail.argtypes = [C.c_long]
        from paper_2302_09708_amd import chefsi
        self.cs = chefsi
        self.dtype = np.float64 if precision == chefsi.FP64 else np.float32
        self.prob = prob
        self.h = chefsi.Handle(prob, precision=precision, max_ns=max_ns)
        self.lib = chefsi.load()

    def status(self, call):
        """The status of a call of the binding (0: it returned)."""
        try:
            call()
        except self.cs.ChefsiError as e:
            return e.status
        return 0

    def kernels(self, what, ns):
        """Names of the kernels of one call ("apply", "filter" or "project") on ns orbitals, in order."""
        size = self.h.chefsi_workspace_bytes(ns)
        if what == "project":  # launches alone: nothing reads or writes the blocks
            a = C.c_void_p(1 << 20)
            self.stub.stub_clear()
            st = self.lib.chefsi_project(self.h.h, a, ns, a, a, a, C.c_size_t(size), None)
            assert st == 0, st
            return self.stub.stub_launches().decode().split()
        ws = np.zeros(size + 256, dtype=np.uint8)
        ws = ws[-ws.ctypes.data % 256:][:size]
        X, Y = (np.zeros((ns, self.prob.nd), dtype=self.dtype) for _ in range(2))
        p, w = (lambda a: C.c_void_p(a.ctypes.data)), C.c_size_t(size)
        self.stub.stub_clear()
        if what == "apply":
            st = self.lib.chefsi_apply_h(self.h.h, p(X), p(Y), ns, p(ws), w, None)
        else:
            lo, cut, hi = self.h.chefsi_spectral_bounds()
            st = self.lib.chefsi_filter(self.h.h, p(X), ns, 3, C.c_double(lo), C.c_double(cut), C.c_double(hi), p(ws), w, None)
        assert st == 0, st
        return self.stub.stub_launches().decode().split()
