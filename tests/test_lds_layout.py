"""LDS areas that a kernel lays out by hand start at the alignment of what they hold.

The dynamic LDS of a workgroup is 16-byte aligned; the resolve phase puts its table of uint2 right behind ResolveLds, whose
size is therefore checked (by the compiler, in a translation unit that sees the kernels' source)."""
import os
import shutil
import subprocess

import pytest

from paper_2005_13789_amd import build as ne_build

SRC = """
#include "{src}"
static_assert(sizeof(ResolveLds) % alignof(uint2) == 0, "the resolve table's slots are read and written whole");
static_assert(alignof(ResolveLds) <= 16, "dynamic LDS");
"""


def test_resolve_table_is_aligned(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    tu = tmp_path / "layout.hip"
    tu.write_text(SRC.format(src=ne_build.SRCS[0]))
    flags = [f for f in ne_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    r = subprocess.run(["hipcc", *flags, "-I", os.path.dirname(ne_build.SRCS[0]), "--offload-host-only", "-fsyntax-only", str(tu)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
