"""The device's square roots, reciprocals and quotients (mhd_physics.hpp), with
hardware estimates as bad as one part in 2^23: the refinement alone has to give
the rounding that the header states.

Bounds: a correctly rounded result is within 0.5 ulp, and what the chains add to
that is the estimate's error to the third power (2^-69, 2e-5 ulp) or times the
46 bits of an intermediate; mrsqrt rounds a product and a sum more, each half an
ulp at most of the result, on top of the final rounding's half: below 1."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_05240_amd", "csrc")


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path_factory.mktemp("chain_probe") / "chain_probe"
    subprocess.run([gxx, "-O1", "-std=c++17", "-ffp-contract=off", "-I", CSRC, "-o", str(exe),
                    os.path.join(HERE, "physics_check", "chain_probe.cpp")], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [[float(x) for x in line.split()] for line in out.splitlines()]


@pytest.mark.parametrize("magnitudes", [0, 1, 2])
def test_chains_round_as_stated(rows, magnitudes):
    root, reciprocal_root, reciprocal, quotient = rows[magnitudes]
    assert root <= 0.5001 and reciprocal <= 0.5001 and quotient <= 0.5001
    assert reciprocal_root <= 1.0


def test_roots_of_the_smallest_normal_numbers(rows):
    """The residual of such a root is subnormal: an ulp, no more."""
    assert rows[3][0] <= 1.0


def test_special_arguments(rows):
    assert rows[4] == [0.0, 1.0, 0.0]
