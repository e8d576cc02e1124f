"""The hardware's reciprocal and square root are at most one bit pattern from the correctly
rounded ones, over every operand for which the BF16 commit's bracketed step and the short
exact square root rely on it (tests/native/hw_approx.hip)."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu


def test_at_most_one_bit_pattern_off():
    exe = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "hw_approx")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    print(r.stdout)
    rows = {name: [int(x) for x in rest] for name, *rest in (line.split() for line in r.stdout.splitlines())}
    assert rows["v_rcp_f32"][0] == 152 << 23 and rows["v_sqrt_f32"][0] == 0x7F800000 - 0x0F800000
    for name, (operands, low, high, far) in rows.items():
        assert far == 0, name
        assert 0 < low + high < operands // 4, name  # (they are approximations)
