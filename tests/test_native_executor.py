"""The serving scheduler's promises to its round executor (no GPU):
tests/native/executor_check.cpp, built plainly and under the sanitizers."""
import os

import pytest

from tests.test_native_sanitizers import CSRC, NATIVE, VARIANTS, _need, _run


@pytest.mark.parametrize("variant", sorted(VARIANTS))
def test_executor_contract(tmp_path, variant):
    cxx, _, flags = VARIANTS[variant]
    _need(cxx)
    exe = str(tmp_path / "executor_check")
    _run([cxx, "-std=c++17", "-Wall", "-Wextra", *flags, "-pthread", "-I", CSRC,
          os.path.join(NATIVE, "executor_check.cpp"), os.path.join(CSRC, "tc_sched.cpp"), "-o", exe])
    r = _run([exe], timeout=120, env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1 second_deadlock_stack=1"))
    assert "all executor checks passed" in r.stdout
    assert "ThreadSanitizer" not in r.stderr and "ERROR" not in r.stderr, r.stderr[-4000:]
