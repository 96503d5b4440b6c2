"""CPU checks of the build: launch shapes that a kernel cannot serve do not compile."""
import os
import subprocess

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
