"""The library's host shell under AddressSanitizer and UndefinedBehaviorSanitizer (host code only; device code is built
as usual).  paper_2604_26555_amd/build.py:build_host_checked compiles csrc/som_api.hip with both sanitizers, links it
with the ordinary objects into libsom_hostsan.so and builds tests/host_shell_check.cpp against it; the driver exits
non-zero on a failed expectation, and a sanitizer report ends it with an error of its own.

Without a GPU the driver covers what needs no device (error strings, null contexts, creation on a missing device).  On
the GPU machine it goes on to one context on device 0: streamed epochs from memory and from a file with several reader
threads, the short-file and bad-argument paths, a resident epoch, create / destroy twice."""
import os
import re
import subprocess

import pytest

import stub_library
from paper_2604_26555_amd import build as libbuild

# The sanitizer's allocator serves the device allocations of the HIP runtime too and keeps freed ones in its quarantine, which
# gives its oldest back when it outgrows this size.  After the HIP runtime has been unloaded it cannot give a device
# allocation back and ends the program ("dev_runtime_unloaded_"), and the runtime's own small deletes on the way out are
# enough to set that off.  The driver's device buffers and the runtime's together come to about the default size of 256 MB,
# so the quarantine is made large enough to hold everything a run frees: nothing leaves it, at exit or before.
QUARANTINE_MB = 4096
ENV = dict(os.environ, ASAN_OPTIONS=f"detect_leaks=0:protect_shadow_gap=0:abort_on_error=0:quarantine_size_mb={QUARANTINE_MB}",
           UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")


def run_driver(*args, timeout):
    r = subprocess.run([libbuild.HOST_CHECKED_DRIVER, *args], env=ENV, capture_output=True, text=True, timeout=timeout)
    print(r.stdout[-2000:], r.stderr[-6000:], flush=True)
    assert r.returncode == 0, f"host_shell_check {' '.join(args)} ended with status {r.returncode}"
    assert "host_shell_check: ok" in r.stdout
    assert "ERROR: AddressSanitizer" not in r.stderr and "runtime error:" not in r.stderr


def test_host_shell_without_a_device():
    objs = [os.path.join(libbuild.HERE, "_build", s.replace(".hip", ".o")) for s in libbuild.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        libbuild.build(verbose=False)
    libbuild.build_host_checked(verbose=False)
    run_driver(timeout=60)


def test_quarantine_holds_what_the_driver_frees(tmp_path):
    """What the driver and its contexts free over a whole run (counted with a HIP runtime that only counts), the driver's
    host copy of the samples, and what the real runtime frees of its own (a run that outgrew 256 MB puts that at 90 MB or
    more), four times over."""
    lib = stub_library.link(str(tmp_path))
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", *stub_library.INCLUDES, os.path.join(stub_library.ROOT, "tests", "host_shell_check.cpp"),
                    "-o", exe, lib, f"-Wl,-rpath,{tmp_path}"], check=True)
    r = subprocess.run([exe, "--device"], env=dict(os.environ, STUB_REPORT="1"), capture_output=True, text=True, timeout=60)
    freed = int(re.search(r"(\d+) freed", r.stderr).group(1))
    print(r.stderr.strip()[-300:])
    assert freed > 100 << 20                       # the count is of the whole run
    assert 4 * (freed + (700_000 * 8 * 4) + (90 << 20)) < QUARANTINE_MB << 20


@pytest.mark.gpu
def test_host_shell_on_the_device():
    if not os.path.exists(libbuild.HOST_CHECKED_DRIVER):
        pytest.skip("the instrumented driver has not been built (__graft_entry__.build() builds it)")
    run_driver("--device", timeout=110)
