"""The shortened division by the smooth scales (activation quantisation) equals the IEEE division for
every pair of significands it can meet: all 11-bit ones of FP16 over all 24-bit ones of FP32."""
import os
import subprocess

import pytest

SOURCE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "short_division.c")


def test_short_division_is_the_ieee_division(tmp_path):
    with open("/proc/cpuinfo") as f:
        flags = f.read()
    if " fma" not in flags or " avx2" not in flags:
        pytest.skip("needs a CPU with FMA instructions")
    exe = tmp_path / "short_division"
    subprocess.run(["gcc", "-O3", "-mavx2", "-mfma", "-ffp-contract=off", "-o", str(exe), SOURCE], check=True, timeout=120)
    out = subprocess.run([str(exe), "1"], check=True, capture_output=True, text=True, timeout=600).stdout
    tried, differ = (int(v) for v in out.split())
    assert tried == (1 << 23) * 1024
    assert differ == 0
