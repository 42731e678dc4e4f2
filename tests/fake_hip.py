"""Runs a piece of Python in a process of its own whose libdsn.so talks to the
HIP runtime of fake_hip.cpp instead of a GPU.  The piece finds: `dsn` (the
binding without torch), `problem(...)` (a handle), `solve(...)` (status and
the report of a solve), `fake` (the fake_* calls) and `events()`."""
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_lib = None

_PRELUDE = '''
import ctypes as C, importlib.util, os, sys
import numpy as np
sys.path.insert(0, %(root)r)
from synthetic.workloads import SourceSpec, random_small_problem
spec = importlib.util.spec_from_file_location("dsn", os.path.join(%(root)r, "paper_1910_11335_amd", "dsn.py"))
dsn = importlib.util.module_from_spec(spec)
spec.loader.exec_module(dsn)
fake = C.CDLL(%(lib)r)
fake.fake_host_limit.argtypes = [C.c_size_t]
fake.fake_capture.argtypes = [C.c_void_p, C.c_int]
fake.fake_events.restype = C.c_char_p
def events():
    return fake.fake_events().decode().split("\\n")[:-1]
def problem(n, sn, precision="fp32", G=1, **kw):
    return dsn.Problem(random_small_problem(1, n=n, sn=sn, L=1, G=G, **kw), precision)
def solve(h, n_src=1, iters=2, combine=False, stream=0):
    src = SourceSpec(position=(-2.3, 0.7, 0.9), spectrum=np.ones(h.G))
    made = [dsn._source_struct(src, h.G) for _ in range(n_src)]
    arr = (dsn.Source * n_src)(*[m[0] for m in made])
    out = np.zeros(8)  # never written: no kernel runs
    o, keep = dsn._opts(h.G, 1e-5, 100, None if iters is None else [iters] * h.G, False, stream, combine=combine)
    info = dsn.SolveInfo()
    st = dsn.lib().dsn_solve(h.handle, arr, n_src, C.byref(o), out.ctypes.data_as(C.c_void_p), None, C.byref(info))
    return st, info
'''


def run(code, timeout=120):
    """The output of `code`; an assertion in it, or a crash, fails the test."""
    global _lib
    if _lib is None:
        tmp = tempfile.TemporaryDirectory(prefix="fake_hip")
        so = os.path.join(tmp.name, "libfake_hip.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", "/opt/rocm/include",
                               os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so])
        _lib = (tmp, so)
    prelude = _PRELUDE % dict(root=ROOT, lib=_lib[1])
    other = [x for x in [os.environ.get("LD_PRELOAD")] if x]
    r = subprocess.run([sys.executable, "-X", "faulthandler", "-c", prelude + code], capture_output=True, text=True, timeout=timeout,
                       env=dict(os.environ, LD_PRELOAD=":".join([_lib[1]] + other), OMP_NUM_THREADS="1"))
    assert r.returncode == 0, "exit %d\n%s%s" % (r.returncode, r.stdout, r.stderr[-3000:])
    return r.stdout
