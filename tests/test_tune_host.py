"""The tile choice by measurement (rs_tune.h) on a simulated device whose clock
falls as it warms up (tests/csrc/tune_host_test.cpp).  No GPU."""
import shutil

import pytest

from host_util import run_host_test


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_tune_pick(tmp_path):
    run_host_test("tune_host_test", tmp_path)
