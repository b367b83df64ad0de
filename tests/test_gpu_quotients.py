"""The quotient from a reciprocal against the IEEE division (a native program
built with the library's flags): every mantissa of the divisor."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu


def test_quotient_from_a_reciprocal_is_the_division():
    exe = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "_bin", "quotient_check")
    assert os.path.exists(exe), "tests/native programs are not built (run __graft_entry__.build())"
    print("[gpu] quotient_check", flush=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    print(r.stdout.strip(), flush=True)
    sys.stdout.flush()
    assert r.returncode == 0 and "mismatches 0" in r.stdout, r.stdout + r.stderr
