"""CPU checks of the build: launch shapes that a kernel cannot serve do not
compile, and the package needs no more than the HIP library."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2211_06934_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

needs_hipcc = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")


def _check(source, *defines):
    """The compiler's verdict on one source (host pass, syntax and templates only)."""
    return subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only", "-std=c++17", "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, *["-D" + d for d in defines],
                           os.path.join(CSRC, source)], capture_output=True, text=True, timeout=300)


@needs_hipcc
def test_flat_kernels_refuse_workgroups_without_the_head_lanes():
    # the last workgroup moves a misaligned buffer's first elements in lanes
    # 64..94: a workgroup of one wave would leave them out
    assert _check("adam.hip").returncode == 0
    for macro in ("SMALL_BLOCK", "UFWD_BLOCK", "UBWD_BLOCK", "URBWD_BLOCK", "URBWD_BLOCK_LONG"):
        bad = _check("adam.hip", "DIFFOPT_%s=64" % macro)
        assert bad.returncode != 0 and "head" in bad.stderr, macro


@needs_hipcc
@pytest.mark.parametrize("source", ["adam.hip", "es.hip", "optim.hip", "treemap.hip"])
def test_wide_accesses_promise_no_more_than_four_byte_alignment(source):
    # buffers and leaves start at any 4-byte aligned address: no 128-bit access
    # may go through a type that tells the compiler 16 bytes
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only", "-std=c++17",
                          "-Werror=align-mismatch", "-Werror=cast-align", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                          os.path.join(CSRC, source)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]


@pytest.mark.parametrize("binding", [None, b"not a library"])
def test_package_runs_on_the_library_alone(tmp_path, binding):
    # without a usable native binding (not built, or built against another
    # torch) every call takes the ctypes path, with the same checks
    pkg = os.path.join(ROOT, "paper_2211_06934_amd")
    shutil.copytree(pkg, tmp_path / "paper_2211_06934_amd",
                    ignore=shutil.ignore_patterns("_binding.so*", "csrc", "__pycache__"))
    if binding is not None:
        (tmp_path / "paper_2211_06934_amd" / "_binding.so").write_bytes(binding)
    code = """
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import paper_2211_06934_amd as P
assert any("native binding" in str(w.message) for w in seen), seen
import torch
x = [torch.ones(8) for _ in range(7)]
h = (0, 1e-3, 0.9, 0.999, 1e-8, 0.0)
for call, error, text in (
        (lambda: P.adam_fwd(*x[:4], *h, *x[4:], stream=0), ValueError, "device memory"),
        (lambda: P.adam_fwd(*[64] * 4, 0, 1e-3, 1.0, 0.999, 1e-8, 0.0, *[64] * 3, stream=0, n=8), P.DiffoptError, "b1 must be in"),
        (lambda: P.es_perturb(x[0], x[1], 0.1, False, x[2], stream=0), ValueError, "device memory")):
    try:
        call()
    except error as e:
        assert text in str(e), e
    else:
        raise AssertionError(text)
P.adam_fwd(*[0] * 4, *h, *[0] * 3, stream=0, n=0)
"""
    env = dict(os.environ, PYTHONPATH=str(tmp_path))
    run = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env=env, capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stderr
