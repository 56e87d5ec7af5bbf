"""The library's host code on a machine without a GPU: the objects of the ordinary build linked with
tests/hip_runtime_stub.cpp instead of the HIP runtime, so that a call notes the kernels it would launch and runs none.
Used to check which path a call takes, what it allocates, and what it does when an allocation fails."""
import ctypes as C
import os
import subprocess

from paper_2604_26555_amd import build as libbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INCLUDES = ["-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include")]


def link(directory) -> str:
    """Builds the stubbed library in `directory`; returns its path."""
    objs = [os.path.join(libbuild.HERE, "_build", s.replace(".hip", ".o")) for s in libbuild.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        libbuild.build(verbose=False)
    stub, lib = os.path.join(directory, "stub.o"), os.path.join(directory, "libsom_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-w", *INCLUDES, "-c",
                    os.path.join(ROOT, "tests", "hip_runtime_stub.cpp"), "-o", stub], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *objs, stub, "-o", lib], check=True)
    return lib


class StubContext:
    """One context of the stubbed library.  Every call returns (return code, [kernel names in launch order])."""

    def __init__(self, path: str, stream=None, device=0):
        self.lib = C.CDLL(path)
        for name in ("stub_allocated", "stub_freed", "stub_peak"):
            getattr(self.lib, name).restype = C.c_size_t
        self.lib.stub_launches.restype = C.c_char_p
        self.lib.stub_limit.argtypes = self.lib.stub_taken.argtypes = [C.c_size_t]
        self.lib.som_last_error.restype = C.c_char_p
        self.lib.som_last_error.argtypes = [C.c_void_p]
        self._buf = C.create_string_buffer(4096)          # stands for every array: no kernel runs, nothing is read
        self._p = C.c_void_p(C.addressof(self._buf))
        self.ctx = C.c_void_p()
        assert self.lib.som_create(C.byref(self.ctx), C.c_int(device), C.c_void_p(stream)) == 0

    def close(self):
        self.lib.som_destroy(self.ctx)

    def switch(self, name, value):
        assert getattr(self.lib, name)(self.ctx, C.c_int(value)) == 0

    def capturing(self, on):
        self.lib.stub_capturing(C.c_int(int(on)))

    def fail(self, kernel=""):
        """Launches of kernels whose name starts with this fail from here on (empty: none does)."""
        self.lib.stub_fail(C.c_char_p(kernel.encode()))

    def limit(self, nbytes=None):
        """Allocations above nbytes fail from here on (None: none does)."""
        self.lib.stub_limit(C.c_size_t(nbytes if nbytes is not None else 2 ** 64 - 1))

    def in_use(self) -> int:
        """Bytes that are allocated now, by every context."""
        return self.lib.stub_allocated() - self.lib.stub_freed()

    def error(self) -> str:
        return self.lib.som_last_error(self.ctx).decode()

    def _run(self, f, *args):
        before = len(self.lib.stub_launches())
        rc = f(self.ctx, *args)
        lines = self.lib.stub_launches()[before:].decode().splitlines()
        self.launches = [(w[0], *map(int, w[1:])) for w in (line.split() for line in lines)]
        return rc, [w[0] for w in self.launches]

    def bmu(self, m, K, D, d2=False, qe=False):
        i64, i32, p = C.c_int64, C.c_int32, self._p
        return self._run(self.lib.som_bmu, p, i64(m), i32(D), i64(D), None, i64(m), p, i32(K), p, p if d2 else None, p if qe else None)

    def accumulate(self, m, K, D, zero_first=True, ldx=None):
        i64, i32, p = C.c_int64, C.c_int32, self._p
        return self._run(self.lib.som_accumulate, p, i64(m), i32(D), i64(ldx or D), None, i64(m), p, i32(K), p, p, C.c_int(int(zero_first)))

    def epoch(self, m, K, D):
        i64, i32, f64, p = C.c_int64, C.c_int32, C.c_double, self._p
        return self._run(self.lib.som_epoch, p, i64(m), i32(D), i64(D), None, i64(m), p, i32(K), p, f64(2.0), C.c_int(0), f64(0.0), None)
