"""The bracketed step of the BF16-state commit, checked on the CPU: wherever the two
ends agree and its ranges hold, the result is the exact form's, for every hardware root
and reciprocal within one bit pattern of the correctly rounded one
(tests/native/bf16_step.c).  A bracket too narrow for the roundings is found out."""
import os
import subprocess

import pytest


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = tmp_path_factory.mktemp("bf16_step") / "bf16_step"
    subprocess.run(["gcc", "-O2", "-std=c11", "-ffp-contract=off", "-mfma", "-o", str(out),
                    os.path.join(root, "tests", "native", "bf16_step.c"), "-lm"], check=True)
    return str(out)


@pytest.mark.parametrize("bits,right", [(20, True), (23, False)])
def test_an_accepted_bracket_holds_the_exact_result(exe, bits, right):
    r = subprocess.run([exe, str(bits)], capture_output=True, text=True, timeout=600)
    checked, accepted, usual, wrong = (int(x) for x in r.stdout.split())
    assert checked > 9 * 10_000_000 and accepted > checked // 4
    assert usual > 0.99 * 9 * 4_000_000  # the form is the usual one on a training shard
    assert (wrong == 0) == right
