"""The chunk pass's LDS layout: every FP64 array starts on an 8-byte boundary
and the whole fits a CU's 160 KB (compiled against the library's header, no
device call)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "efem_internal.h"
using namespace efem;
static_assert((5 * kPieceBytes) % 8 == 0, "nodal sums");
static_assert((5 * kPieceBytes + kChunkCap * 24) % 8 == 0, "wave sums, over the staging words");
static_assert(kChunkLds % 8 == 0, "shares of v.K v");
static_assert(kChunkLds + kChunkPqLds <= 160 * 1024, "one CU's LDS");
"""


def test_fp64_arrays_are_aligned(tmp_path):
    src = tmp_path / "layout.cpp"
    src.write_text(SOURCE)
    res = subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-fsyntax-only", "-I", os.path.join(ROOT, "include"),
                          "-I", os.path.join(ROOT, "paper_2602_12365_amd", "csrc"), str(src)],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
