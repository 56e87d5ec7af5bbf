"""CPU-side checks of the boundary: the library loads, exports what include/som.h declares, fails loudly."""
import ctypes
import os
import re

import pytest

import paper_2604_26555_amd as pkg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "som.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(som_[a-z_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(pkg.LIB_PATH):
        from paper_2604_26555_amd.build import build
        build(verbose=False)
    return pkg.load_library()


def test_header_and_binding_agree():
    assert _declared() == sorted(pkg.EXPORTS)


def test_library_exports_every_declared_symbol(lib):
    for name in _declared():
        assert hasattr(lib, name), name


def test_strerror_without_gpu(lib):
    assert lib.som_strerror(0) == b"ok"
    assert lib.som_strerror(pkg.SOM_EINVAL) == b"invalid argument"
    assert lib.som_strerror(-99) == b"unknown error code"
    assert lib.som_last_error(None) == b"null context"


def test_no_cpu_fallback(lib):
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    handle = ctypes.c_void_p()
    assert lib.som_create(ctypes.byref(handle), 0, None) == pkg.SOM_ESTATE
    assert not handle.value
    with pytest.raises(RuntimeError):
        pkg.Som(0)
    assert lib.som_sync(None) == pkg.SOM_EINVAL


def test_product_never_imports_the_oracle():
    for dirpath, _, files in os.walk(os.path.join(ROOT, "paper_2604_26555_amd")):
        for f in files:
            if f.endswith((".py", ".hip", ".hpp", ".h")):
                src = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in src, os.path.join(dirpath, f)


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU; asked for more it says so and exits instead of printing a number."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "one GPU" in (r.stdout + r.stderr) and "{" not in r.stdout


def test_nothing_committed_points_at_the_working_folder():
    """Probes and helper scripts live in a git-ignored working folder; no committed source may import, read or run them."""
    import subprocess
    tracked = subprocess.run(["git", "ls-files"], cwd=ROOT, capture_output=True, text=True).stdout.split()
    if not tracked:
        pytest.skip("not a git checkout")
    needle = "_" + "work/"
    for f in tracked:
        reviews = ("VERDICT.md", "ADVICE.md", "SURVEY.md", "BASELINE.md", "BASELINE.json")      # not this build's own files
        record = re.fullmatch(r"[A-Z]+_r\d+\.json", f)        # nor are the records of benchmark and test runs (BENCH_r01.json ...)
        if f.endswith((".py", ".hip", ".hpp", ".h", ".cpp", ".md", ".json")) and f not in reviews and not record:
            assert needle not in open(os.path.join(ROOT, f), errors="ignore").read(), f


def test_assembly_names_the_registers_it_writes():
    """An inline-assembly statement that writes m0 must say so, or the compiler may keep a value of its own there."""
    found = 0
    csrc = os.path.join(ROOT, "paper_2604_26555_amd", "csrc")
    for f in sorted(os.listdir(csrc)):
        for asm in re.findall(r"\basm\s+(?:volatile\s*)?\((.*?)\);", open(os.path.join(csrc, f)).read(), flags=re.S):
            template = asm.split('" :')[0]
            if re.search(r"\bm0\b", template):
                found += 1
                assert re.search(r'"m0"', asm), f"{f}: {asm.strip()[:120]}"
    assert found >= 1
