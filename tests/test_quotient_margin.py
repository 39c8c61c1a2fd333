"""How near a half-integer the row quantisers' shortcut has to leave a quotient to the division: its arithmetic on the host, for every
fp16 value up to every fp16 row maximum, against the definition.  (The kernels themselves: test_gpu_rowwise.py.)"""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "..", "paper_2311_09550_amd", "csrc", "common.hpp")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    (margin, rest), = re.findall(r"constexpr float kTieMargin = (\S+), kTieRest = (\S+);", open(SOURCE, encoding="utf-8").read())
    exe = str(tmp_path_factory.mktemp("margin") / "quotient_margin")
    subprocess.run(["gcc", "-O2", "-std=c11", "-ffp-contract=off", "-fopenmp", f"-DTIE_MARGIN={margin}", f"-DTIE_REST={rest}",
                    os.path.join(HERE, "quotient_margin.c"), "-o", exe, "-lm"], check=True)
    return exe


def _run(program, *args):
    return map(int, subprocess.run([program, *map(str, args)], check=True, capture_output=True, text=True).stdout.split())


# Of all pairs 7.7e-6 are sent to the division for 127 beside the exact half-integers, and none for 7; a band of 1e-4, as it was before
# the margins followed from the arithmetic, would send 6.6e-5.
@pytest.mark.parametrize("qmax", [127, 7])
def test_no_code_is_wrong_and_few_values_are_sent_to_the_division(program, qmax):
    pairs, halves, wrong, wrong_per_value, sent, sent_per_value = _run(program, qmax, 1, 1)
    assert pairs == 0x7BFF * 0x7C00 // 2 + 0x7BFF and wrong == 0 and wrong_per_value == 0
    assert halves <= sent_per_value <= sent <= halves + 2e-5 * qmax / 127 * pairs


@pytest.mark.parametrize("first", [1, 31743])
def test_single_row_maxima(program, first):
    pairs, halves, wrong, wrong_per_value, sent, sent_per_value = _run(program, 127, first, 31742)
    assert pairs > 0 and wrong == 0 and wrong_per_value == 0 and sent >= halves and sent_per_value >= halves
