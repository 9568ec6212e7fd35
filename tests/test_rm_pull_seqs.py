"""CPU check of the sequences whose values the best responses pull
(tests/cpp/rm_pull_seqs_check.cpp, compiled with g++ together with the
library's host builder): sequence numbers are kept whole, also past 24 bits
(one-card games of many bets reach them)."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def helper(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("pulls") / "libpulls.so")
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2112_03804_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "rm_pull_seqs_check.cpp"),
                    os.path.join(ROOT, "paper_2112_03804_amd", "csrc", "host_build.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("first", [3, (1 << 24) - 8, 1 << 24, (1 << 29) + 5])
def test_pulled_sequences_are_whole(helper, first):
    assert helper.check_rm_pull_seqs(first) == 0
