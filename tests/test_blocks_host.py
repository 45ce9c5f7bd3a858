"""The workspaces that plans keep for their allocating calls (rs_blocks.h), on a
device of the test's own (tests/csrc/blocks_host_test.cpp): bounds, streams that
never come back, short memory, threads.  No GPU."""
import shutil

import pytest

from host_util import run_host_test


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("sanitizers", ["address,undefined", "thread"])
def test_kept_blocks(tmp_path, sanitizers):
    run_host_test("blocks_host_test", tmp_path, sanitizers)
