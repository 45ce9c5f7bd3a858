"""The chunk rule of the plans (rs_chunks.h), swept on the CPU by
tests/csrc/chunks_host_test.cpp, built with g++ under AddressSanitizer and
UndefinedBehaviorSanitizer.  No GPU."""
import shutil

import pytest

from host_util import run_host_test


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_chunk_rule(tmp_path):
    run_host_test("chunks_host_test", tmp_path)
