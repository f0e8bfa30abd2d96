"""The biased 64-bit sums of the matrix-core kernels leave int64_t on ordinary values: formed with
checks of signed overflow on the host they raise none, and give exact residues."""
import os
import subprocess

import pytest

from synth import Q2_DEFAULT, Q_DEFAULT

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("Q", [Q_DEFAULT, Q2_DEFAULT, 12289, 1073692673])
def test_biased_sums(tmp_path, Q):
    exe = str(tmp_path / "wrap64")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=signed-integer-overflow", "-fno-sanitize-recover=all",
                    "-I" + os.path.join(ROOT, "paper_2310_12441_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "wrap64.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe, str(Q)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr
