"""LDS areas that a kernel lays out by hand start at the alignment of what they hold.

The dynamic LDS of a workgroup is 16-byte aligned; the resolve phase puts its table of uint2, which it clears two slots at a time,
right behind ResolveLds, whose size is therefore checked (by the compiler, in a translation unit that sees the kernels' source)."""
import os
import shutil
import subprocess

import pytest

from paper_2005_13789_amd import build as ne_build

SRC = """
#include "{src}"
static_assert(sizeof(ResolveLds) % alignof(uint4) == 0, "the resolve table is cleared two slots at a time");
static_assert(alignof(ResolveLds) <= 16, "dynamic LDS");
"""


def syntax_check(tmp_path, source):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    tu = tmp_path / "layout.hip"
    tu.write_text(source.format(src=ne_build.SRCS[0]))
    flags = [f for f in ne_build.HIPCC_FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    r = subprocess.run(["hipcc", *flags, "-I", os.path.dirname(ne_build.SRCS[0]), "--offload-host-only", "-fsyntax-only", str(tu)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]


def test_resolve_table_is_aligned(tmp_path):
    syntax_check(tmp_path, SRC)


BINS = """
#include "{src}"
constexpr Binning a = binning(2 * 2100), b = binning(2 * 60000);
static_assert(a.bits == 6 && a.tile == 2 * 128 && a.tiles == 17 && most_singles(a) >= 60, "2100 pairs");
static_assert(b.bits == 8 && b.tile == 2 * 512 && b.tiles == 118 && most_singles(b) == 18, "60 000 pairs");
static_assert(kShortSegment == 32, "listed entries of a tile");
"""


def test_bins_of_the_batches_that_fill_a_segment(tmp_path):
    """What tests/test_gpu_work_items.py takes for granted of its batches of 2100 and 60 000 pairs without negatives."""
    syntax_check(tmp_path, BINS)
