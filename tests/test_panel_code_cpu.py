"""The code that the compiler makes of the panel kernel: what it waits for, how the waves add up, its LDS."""
import os
import re
import subprocess

import pytest

from paper_2509_01229_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _waits_right_behind_weights(body):
    """The lines where the compiler waits for vector memory behind a load of weights or parameters (buffer loads;
    the scales are global loads) with no wait written by hand in between."""
    found, by_hand, behind_load = [], False, False
    for line in body.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            by_hand = "#ASMSTART" in line
        elif re.match(r"\s*(buffer|global)_load", line):
            behind_load = "buffer_load" in line
        elif re.match(r"\s*s_waitcnt vmcnt", line):
            if behind_load and not by_hand:
                found.append(line.strip())
            behind_load = False
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """The code of 32 x 32 panels by group size ("1": 128), from a source that also states what its LDS must allow."""
    asm = str(tmp_path_factory.mktemp("panel") / "panel.s")
    flags = [f for f in B.FLAGS if f not in ("-shared", "-lpthread", "-Rpass-analysis=kernel-resource-usage")]
    subprocess.run([B.HIPCC, *flags, "-w", "-S", "--cuda-device-only", "-o", asm,
                    os.path.join(ROOT, "tests", "native", "panel_code.hip")], check=True)
    with open(asm) as f:
        text = f.read()
    found = dict(re.findall(r"^_ZN3lqq17w4a8_panel_kernelILi1ELi8ELi1ELb(\d)ELb1EE\S*:(.*?)\.end_amdhsa_kernel", text, re.M | re.S))
    assert set(found) == {"0", "1"}
    return found


def test_weights_and_parameters_are_waited_for_where_they_are_used(kernels):
    """A unit's weights and parameters are loaded two units ahead, and each unit waits for its own by hand.
    Widening the 2 bytes of a lane's parameters (groups of 128) where they are loaded made the compiler wait for
    that load at once, in front of the first unit and at the end of every second one: 3 to 4 % of the time."""
    for body in kernels.values():
        units = body[:body.rindex("v_mfma")]
        assert units.count("buffer_load") >= 9
        assert _waits_right_behind_weights(units) == []


def test_the_waves_sums_are_added_up_without_atomics(kernels):
    """Adding to one copy in LDS with atomics took 5 to 9 % longer with one unit a wave (K up to 1024)."""
    for body in kernels.values():
        assert "ds_add" not in body and "ds_write_b128" in body
