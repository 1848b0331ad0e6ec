"""Runs a function of a test module in a child process in which libmt.so works on
the host-memory HIP runtime of hip_host_stub.cpp: the library's host code (loaders,
launch dispatch, workspaces, tuner) without a GPU.  Kernels do not run."""
import ctypes as C
import dataclasses
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "hip_host_stub.cpp")
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


def build(folder) -> str:
    lib = os.path.join(str(folder), "libhip_host_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I", HIP_INCLUDE, SRC, "-o", lib], check=True)
    return lib


def run(lib, module, function, *args):
    """module.function(stub, *args) in a child process; raises if it fails."""
    code = (f"import sys; sys.path.insert(0, {ROOT!r})\n"
            "from tests import _host_stub\n"
            f"stub = _host_stub.Stub({lib!r})\n"
            f"import {module}\n{module}.{function}(stub, *{args!r})\nprint('child ok')\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=ROOT,
                       timeout=300)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]


@dataclasses.dataclass
class Launch:
    name: str
    grid: int
    block: int
    lds: int
    tables_live: bool


class Stub:
    def __init__(self, lib):
        self.c = C.CDLL(lib, mode=C.RTLD_GLOBAL)
        self.c.stub_limit.argtypes = [C.c_size_t]
        self.c.stub_used.restype = self.c.stub_peak.restype = C.c_size_t
        self.c.stub_cheap.argtypes = [C.c_char_p]
        self.c.stub_launch.restype = C.c_char_p
        self.c.stub_launch.argtypes = [C.c_int, C.POINTER(C.c_uint), C.POINTER(C.c_uint),
                                       C.POINTER(C.c_size_t), C.POINTER(C.c_int)]
        from paper_2512_10520_amd import _lib
        self.m = _lib
        self.L = _lib.load()

    def launches(self):
        out = []
        for i in range(self.c.stub_launches()):
            g, b, s, v = C.c_uint(), C.c_uint(), C.c_size_t(), C.c_int()
            n = self.c.stub_launch(i, C.byref(g), C.byref(b), C.byref(s), C.byref(v))
            out.append(Launch(n.decode(), g.value, b.value, s.value, bool(v.value)))
        self.c.stub_clear()
        return out

    # loaders on workloads' objects; each returns the status code
    def histograms(self, h):
        import numpy as np
        e, c = np.ascontiguousarray(h.p_edges, np.float64), np.ascontiguousarray(h.counts, np.uint32)
        return self.L.mt_load_histograms(c.shape[0], c.shape[1], e.ctypes.data, c.shape[2],
                                         h.loss_lo, h.loss_hi, c.shape[3], h.scat_lo, h.scat_hi,
                                         c.ctypes.data)

    def geometry(self, g):
        import numpy as np
        mat = np.ascontiguousarray(g.material, np.int32)
        bb = np.ascontiguousarray(g.b_box, np.float32)
        mag = np.ascontiguousarray(g.magnet, np.int32)
        world = np.ascontiguousarray(g.world, np.float64)
        vol = np.ascontiguousarray(g.box if g.poly is None else g.poly, np.float64)
        fn = self.L.mt_load_geometry if g.poly is None else self.L.mt_load_blocks
        return fn(len(mat), vol.ctypes.data, mat.ctypes.data, bb.ctypes.data, mag.ctypes.data,
                  g.n_mag, world.ctypes.data)

    def field(self, b):
        import numpy as np
        b = np.ascontiguousarray(b, np.float32)
        lo, hi = np.zeros(3), np.ones(3)
        return self.L.mt_load_field(b.shape[2], b.shape[1], b.shape[0], lo.ctypes.data,
                                    hi.ctypes.data, b.ctypes.data)

    def params(self, **kw):
        p = self.m.MtParams(step_m=0.02, max_steps=1000, p_min=0.2, n_variants=1, r_scale=1.0)
        for k, v in kw.items():
            setattr(p, k, v)
        return p

    def _arrays(self, n):
        p = C.c_void_p(4096)             # never read: kernels do not run
        return self.m.MtMuons(p, p, p, p, p, p, p), self.m.MtResult(p, p, p)

    def propagate(self, p, n, noalloc=False):
        m, r = self._arrays(n)
        fn = self.L.mt_propagate_noalloc if noalloc else self.L.mt_propagate
        return fn(C.byref(p), n, C.byref(m), C.byref(m), C.byref(r), None)

    def autotune(self, p, n):
        m, r = self._arrays(n)
        b, c, ms = C.c_int32(), C.c_int32(), C.c_float()
        rc = self.L.mt_autotune(C.byref(p), n, C.byref(m), C.byref(m), C.byref(r), None, C.byref(b),
                                C.byref(c), C.byref(ms))
        return rc, b.value, c.value, ms.value
