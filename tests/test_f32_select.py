"""Which float32 calls the matrix-core kernels take, on the host: the selection is plain C++ (csrc/f32_select.h)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_22275_amd", "csrc")


def _holds(tmp_path, *conditions):
    src = tmp_path / "select.cpp"
    src.write_text('#include "f32_select.h"\nusing namespace vm;\n' +
                   "".join(f"static_assert({c}, \"\");\n" for c in conditions))
    cxx = shutil.which("g++") or shutil.which("amdclang++") or "/opt/rocm/bin/amdclang++"
    r = subprocess.run([cxx, "-std=c++17", "-fsyntax-only", f"-I{CSRC}", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_grids_that_one_launch_holds(tmp_path):
    """A launch has fewer than 2^32 threads in a dimension.  Frames of one token take a tile of 32 rows each: 2^26 of them are
    the limit, and the calls beyond it stay on the kernels with a three-dimensional grid."""
    _holds(tmp_path,
           "grid_fits(0xffffffffLL / 256, 256)", "!grid_fits((1LL << 32) / 256, 256)", "!grid_fits(0, 64)",
           "f32_attend_fits((1LL << 26) - 64, 1)", "!f32_attend_fits(1LL << 26, 1)", "!f32_attend_fits(65535LL * 65535, 1)",
           "f32_attend_fits(1LL << 20, 32 * 63)", "!f32_attend_fits(1LL << 20, 32 * 64)",
           "f32_attend_fits(1, 1)", "f32_attend_fits(1, 0x7fffffffLL - 4096)", "!f32_attend_fits(1, 0x7fffffffLL)")


def test_few_keys(tmp_path):
    """Nearly empty tiles stay on the kernels with a wave per row; any call of one full tile of keys, and few rows over many keys, do
    not."""
    _holds(tmp_path,
           "f32_few_keys(128, true, 8000, 4, 4)", "!f32_few_keys(128, true, 8000, 5, 5)", "f32_few_keys(128, false, 8000, 3, 3)",
           "f32_few_keys(32, false, 8000, 2, 2)", "!f32_few_keys(32, false, 8000, 3, 3)",
           "f32_few_keys(128, true, 100, 12, 12)", "!f32_few_keys(128, true, 100, 17, 17)", "f32_few_keys(128, true, 600, 4, 4)",
           "!f32_few_keys(128, true, 600, 6, 6)", "f32_few_keys(64, false, 100, 4, 4)", "!f32_few_keys(64, false, 4, 13, 13)",
           "!f32_few_keys(128, true, 1, 1, 32)", "!f32_few_keys(64, true, 1, 1, 0x7fffffff)", "!f32_few_keys(32, true, 1, 4, 1000)",
           "f32_few_keys(128, true, 2, 400, 1)", "!f32_few_keys(128, true, 8, 1000, 1)",
           "!f32_few_keys(128, true, 1LL << 31, 1LL << 31, 24)")
