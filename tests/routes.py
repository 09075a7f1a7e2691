"""What a call launches or refuses, without a GPU: the child process loads libsdnn over tests/hip_stub.cpp.

run(code) runs `code` there with these names: sdnn, np, C, Net (below), layer(n_out, n_in, lengths)."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
_built = {}

PRELUDE = '''
import ctypes as C
import numpy as np
from paper_2104_11805_amd import sdnn
lib = sdnn.lib()
stub = C.CDLL(None)                               # the global scope: preloaded
stub.stub_log.restype = C.c_char_p
stub.stub_arg.restype = C.POINTER(C.c_int32)
stub.stub_long_arg.restype = C.POINTER(C.c_uint64)
ADDR = 1 << 40                                     # device addresses: never followed on the host

def layer(n_out, n_in, lengths, bias=None):
    """Row r has lengths[r % len(lengths)] entries in the first columns."""
    deg = np.resize(np.asarray(lengths, np.int32), n_out)
    rp = np.zeros(n_out + 1, np.int32)
    np.cumsum(deg, out=rp[1:])
    ci = (np.arange(rp[-1], dtype=np.int64) - np.repeat(rp[:-1], deg)).astype(np.int32)
    return n_out, n_in, rp, ci, np.ones(ci.size, np.float32), bias

class Net:
    def __init__(self, layers, max_batch, training=False, act_cap=2.0, col_idx=True, **options):
        self.keep = layers
        arr = (sdnn.sdnn_layer * len(layers))()
        for k, (n_out, n_in, rp, ci, va, bi) in enumerate(layers):
            arr[k] = sdnn.sdnn_layer(n_out, n_in, rp.ctypes.data, ci.ctypes.data if col_idx else None, va.ctypes.data,
                                     None if bi is None else bi.ctypes.data)
        self.arr = arr
        opt = dict(update_bias=1, activation=0, fuse_gradient=0, panel_cols=0, reorder_rows=0, lds_forward=0)
        opt.update(options)
        self.cfg = sdnn.sdnn_config(act_cap, max_batch, int(training), *opt.values())
        n = C.c_size_t()
        assert lib.sdnn_workspace_bytes(arr, len(layers), C.byref(self.cfg), C.byref(n)) == 0, sdnn.last_error()
        self.bytes = n.value                          # col_idx=False: sized without the columns
        for k, l in enumerate(layers):
            arr[k].col_idx = l[3].ctypes.data
        self.h = C.c_void_p()
        rc = lib.sdnn_create(arr, len(layers), C.byref(self.cfg), C.c_void_p(ADDR), n, None, C.byref(self.h))
        assert rc == 0, sdnn.last_error()

    def __call__(self, name, *args):
        """(return code, launches) of a call; integers above 2^32 are passed as pointers."""
        stub.stub_clear()
        rc = getattr(lib, name)(self.h, *[C.c_void_p(a) if isinstance(a, int) and a >= 1 << 32 else a for a in args])
        log = [l for l in stub.stub_log().decode().split("\\n") if l]
        return rc, log

X0, XL, DL = 2 << 40, 3 << 40, 4 << 40
'''


def stub():
    """Path of the stand-in runtime, compiled once per test run."""
    if "path" not in _built:
        import tempfile
        _built["dir"] = tempfile.TemporaryDirectory()
        path = os.path.join(_built["dir"].name, "hip_stub.so")
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM + "/include",
                        os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", path], check=True)
        _built["path"] = path
    return _built["path"]


def run(code):
    from paper_2104_11805_amd import sdnn
    sdnn.lib()                                     # built if it is not there
    env = dict(os.environ)
    env["LD_PRELOAD"] = stub() + (" " + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    out = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code)], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    return out.stdout
