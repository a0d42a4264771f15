"""The served results' way to the collecting threads, on the CPU: plain, with
ThreadSanitizer and with AddressSanitizer + UndefinedBehaviorSanitizer
(tests/native/sched_results.cpp)."""
import os

import pytest

from test_native_sanitizers import CLANG, INC, NATIVE, _build_and_run

SOURCE = ["-std=c++17", "-g", "-pthread"] + INC + [os.path.join(NATIVE, "sched_results.cpp")]


@pytest.mark.parametrize("kind", ["plain", "thread", "address"])
def test_results_reach_the_collecting_threads(tmp_path, kind):
    if kind == "thread" and not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not found")
    cmd = {"plain": ["g++", "-O2"],
           "thread": [CLANG, "-O1", "-fsanitize=thread", "-DSANITIZE_THREAD"],
           "address": ["g++", "-O1", "-fsanitize=address,undefined",
                       "-fno-sanitize-recover=all", "-fno-omit-frame-pointer"]}[kind]
    _build_and_run(str(tmp_path), "results", cmd + SOURCE)
