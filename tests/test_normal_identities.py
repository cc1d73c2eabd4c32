"""Exhaustive CPU check of the rearranged Box-Muller arithmetic of the step kernels: the same bits
as the definition that the oracle evaluates, for every Philox word (tests/csrc/normal_identities.c)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_rearranged_normals_match_the_definition(tmp_path):
    exe = str(tmp_path / "normal_identities")
    subprocess.run(["gcc", "-O2", "-ffp-contract=off", "-fno-fast-math",
                    os.path.join(HERE, "csrc", "normal_identities.c"), "-o", exe, "-lm"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "radius mismatches 0, scale mismatches 0, parity mismatches 0, exp mismatches 0" in out.stdout
