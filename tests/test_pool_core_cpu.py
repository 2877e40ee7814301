"""CPU checks of the device memory pool's lists (pool_core.h): built with g++
here, with AddressSanitizer/UBSan and with ThreadSanitizer, run without a GPU."""

from __future__ import annotations

import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "cpp", "pool_core_test.cpp")
INC = os.path.join(ROOT, "paper_1708_04329_amd", "csrc")


@pytest.mark.parametrize("flags", [["-O2"], ["-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer"],
                                   ["-O1", "-g", "-fsanitize=thread"]])
def test_pool_core(flags):
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "t")
        subprocess.check_call(["g++", "-std=c++17", "-pthread", *flags, "-I", INC, SRC, "-o", exe])
        out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert out.returncode == 0, out.stderr
        assert out.stdout.strip() == "OK"
