"""The code that the compiler makes of the panel kernel: what it waits for."""
import os
import re
import subprocess

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


def test_weights_and_parameters_are_waited_for_where_they_are_used(tmp_path):
    """A unit's weights and parameters are loaded two units ahead, and each unit waits for its own by hand.
    Widening the 2 bytes of a lane's parameters (groups of 128) where they are loaded made the compiler wait for
    that load at once, in front of the first unit and at the end of every second one: 3 to 4 % of the time."""
    asm = str(tmp_path / "panel.s")
    flags = [f for f in B.FLAGS if f not in ("-shared", "-lpthread", "-Rpass-analysis=kernel-resource-usage")]
    subprocess.run([B.HIPCC, *flags, "-w", "-S", "--cuda-device-only", "-o", asm,
                    os.path.join(ROOT, "tests", "native", "panel_code.hip")], check=True)
    with open(asm) as f:
        text = f.read()
    kernels = dict(re.findall(r"^_ZN3lqq17w4a8_panel_kernelILi1ELi8ELi1ELb(\d)ELb1EE\S*:(.*?)s_endpgm", text, re.M | re.S))
    assert set(kernels) == {"0", "1"}
    for body in kernels.values():
        assert body.count("buffer_load") >= 9
        assert _waits_right_behind_weights(body) == []
