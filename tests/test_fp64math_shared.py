"""The FP64 power function is checked on the host (tests/sanitize/fp64math_check.hip):
that says something of the GPU's only if both compile the same expressions."""

import os

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_10809_amd", "csrc")


def test_host_and_device_share_every_expression():
    with open(os.path.join(CSRC, "fp64math.hpp")) as fh:
        code = [line.split("//")[0] for line in fh]
    assert not [line for line in code if "DEVICE_COMPILE" in line or "__builtin_amdgcn" in line]
    assert sum("__host__ __device__" in line for line in code) == 3
