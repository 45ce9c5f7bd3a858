"""Paths and workspace layout of the range-Doppler calls (rs_rd_layout.h),
swept on the CPU by tests/csrc/rd_layout_host_test.cpp.  No GPU."""
import shutil

import pytest

from host_util import run_host_test


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rd_layout(tmp_path):
    run_host_test("rd_layout_host_test", tmp_path)
