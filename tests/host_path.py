"""The library's host path without a GPU: ``run(script)`` executes a script in a
child process whose HIP runtime is the stub of hip_stub.cpp, with ``stub``, ``lib``
(the loaded library) and ``Plan`` (a plan made without torch) at hand; the script
leaves its answer in ``out``."""
import json
import os
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = r'''
import ctypes as ct, json, sys
import numpy as np
sys.path.insert(0, {root!r})
from paper_2311_02101_amd import hp, workload as wl
stub = ct.CDLL({stub!r}, mode=ct.RTLD_GLOBAL)
stub.stub_log.restype, stub.stub_bytes.restype = ct.c_char_p, ct.c_size_t
lib = ct.CDLL(hp.LIB_PATH)
lib.hp_last_error.restype = lib.hp_status_string.restype = ct.c_char_p
hp._lib, hp._stream_handle = lib, lambda stream: ct.c_void_p(None)


class Plan(hp.Plan):
    def state(self):
        """A state in host memory; its sweep counter is ``state.t``."""
        nu = np.float32 if self.precision == "f32" else np.float64
        size = self.total_vars * self.B
        self.a = a = [np.zeros(size, np.uint8), np.zeros(size, nu), np.zeros(self.F * self.B, np.int32),
                      np.zeros(size, np.uint8)]
        self.t = np.zeros(1, np.int64)
        return hp.HpState(*[x.ctypes.data for x in a], self.t.ctypes.data, self.total_vars, self.F, self.B,
                          a[1].itemsize)

    def call(self, name, *args):
        return getattr(lib, name)(self._h, *args, ct.c_void_p(None))


def kernels():
    return stub.stub_log().decode().split()


out = None
'''


def _stub(tmp):
    so, attr = os.path.join(tmp, "hip_stub.so"), os.path.join(tmp, "attr.cpp")
    with open(attr, "w") as fh:
        fh.write("#include <hip/hip_runtime_api.h>\n"
                 "extern const int stub_attr_cus;\nconst int stub_attr_cus = hipDeviceAttributeMultiprocessorCount;\n")
    subprocess.run([shutil.which("g++") or "c++", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(ROOT, "tests", "hip_stub.cpp"), attr, "-o", so], check=True)
    return so


def run(tmp, script):
    code = PRELUDE.format(root=ROOT, stub=_stub(str(tmp))) + script + "\nprint('OUT' + json.dumps(out))\n"
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    return json.loads(res.stdout.split("OUT")[-1])
