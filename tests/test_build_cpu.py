"""What the build and the import refuse. Kernels read and write rows at element
alignment, and a load or store that promises the compiler more than that is
undefined, also where today's instructions would take any address. The
binding's two binaries come from one build."""

import importlib.util
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_25442_amd", "csrc")


def _build_module():
    spec = importlib.util.spec_from_file_location("_wb_build", os.path.join(ROOT, "paper_2609_25442_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


B = _build_module()


def _compile(path, *flags):
    return subprocess.run([B.HIPCC, *B.DEVICE_FLAGS, *flags, "-fsyntax-only", path], capture_output=True, text=True)


@pytest.mark.parametrize("source", B.DEVICE_SOURCES)
def test_no_access_promises_more_alignment_than_its_data_has(source):
    r = _compile(os.path.join(CSRC, source), "-Walign-mismatch")
    assert r.returncode == 0 and "align-mismatch" not in r.stderr, r.stderr


def test_the_build_refuses_a_promise_of_alignment(tmp_path):
    # the alignment of a typedef is lost where a template parameter is deduced
    src = tmp_path / "promise.hip"
    src.write_text("""#include <hip/hip_runtime.h>
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef u4 u4_a2 __attribute__((aligned(2)));
template <class T> __device__ T ld(const T* p) { return __builtin_nontemporal_load(p); }
__global__ void k(const char* p, u4* out) { *out = ld(reinterpret_cast<const u4_a2*>(p)); }
""")
    r = _compile(str(src))
    assert r.returncode != 0 and "align-mismatch" in r.stderr, r.stderr


@pytest.mark.parametrize("args", ["missing", "broken"])
def test_import_without_the_argument_checks_names_the_build(args, tmp_path):
    """A tree built before the argument checks came, or a file that does not
    load, says what to run (as a missing library does)."""
    pkg = tmp_path / "paper_2609_25442_amd"
    pkg.mkdir()
    for name in ("__init__.py", "libwb.so"):
        os.symlink(os.path.join(ROOT, "paper_2609_25442_amd", name), pkg / name)
    if args == "broken":
        (pkg / "_args.so").write_bytes(b"no library")
    r = subprocess.run([sys.executable, "-c", "import paper_2609_25442_amd"], cwd=tmp_path, capture_output=True, text=True,
                       env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert r.returncode != 0 and "ImportError" in r.stderr and "paper_2609_25442_amd/build.py" in r.stderr, r.stderr
