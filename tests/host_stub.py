"""The library's host code on the runtime of tests/hip_stub.hip: builds both (host pass only) and
hands out the package's binding on top of them.  Runs without a GPU."""
import ctypes as C
import os
import subprocess
from collections import namedtuple

from paper_2509_04277_amd import rod as R

HERE = os.path.dirname(os.path.abspath(__file__))
REPO = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(REPO, "paper_2509_04277_amd", "csrc")
Launch = namedtuple("Launch", "kernel stream grid")


def build(folder):
    flags = ["--offload-arch=gfx950", "--offload-host-only", "-O1", "-g", "-std=c++17", "-fPIC",
             "-I", os.path.join(REPO, "include"), "-I", CSRC]
    objs = []
    for src in (os.path.join(CSRC, "rod_lib.hip"), os.path.join(HERE, "hip_stub.hip")):
        objs.append(os.path.join(folder, os.path.basename(src) + ".o"))
        subprocess.run([HIPCC, *flags, "-c", src, "-o", objs[-1]], check=True)
    # (symbols bound inside: a HIP runtime in the process is not called; the objects refer to
    # device code that is not there and never asked for)
    undefined = subprocess.run(["nm", "-u", *objs], check=True, capture_output=True, text=True).stdout
    absent = sorted({w for w in undefined.split() if w.startswith("__hip_fatbin")})
    out = os.path.join(folder, "libhost.so")
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs",
                    *("-Wl,--defsym,%s=0" % a for a in absent), *objs, "-o", out, "-lpthread"],
                   check=True)
    return out


class Stub:
    """The loaded pair: ``lib`` for the binding, and what the runtime is told and saw."""

    def __init__(self, path):
        self.lib = C.CDLL(path)
        for name, (res, args) in R._SIGS.items():
            f = getattr(self.lib, name)
            f.restype, f.argtypes = res, args
        for name, args in (("stub_hold", [C.c_void_p, C.c_int]), ("stub_capture", [C.c_void_p, C.c_int]),
                           ("stub_fail_malloc", [C.c_longlong]), ("stub_cost", [C.c_char_p, C.c_double])):
            getattr(self.lib, name).argtypes = args
        self.lib.stub_launch.restype = C.c_char_p
        self.lib.chunk_first_mark.restype = self.lib.chunk_launch_marks.restype = C.c_uint32
        self.lib.chunk_mark_behind.argtypes = [C.c_uint32, C.c_uint32]

    def launches(self, since=0):
        s, g, out = C.c_void_p(), C.c_uint(), []
        for i in range(since, self.lib.stub_launches()):
            name = self.lib.stub_launch(i, C.byref(s), C.byref(g)).decode()
            out.append(Launch(name, s.value or 0, g.value))
        return out
