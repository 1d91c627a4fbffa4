"""The batch tuner's search on made-up times: no plan out of noise or drift, the
faster tile where there is one."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_05240_amd", "csrc")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path_factory.mktemp("tune_probe") / "tune_probe"
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", CSRC, "-o", str(exe),
                    os.path.join(HERE, "physics_check", "tune_probe.cpp")], check=True)

    def run(noise, drift, cls, gain):
        text = "\n".join("%d %g %g %d %g" % (q, noise, drift, cls, gain) for q in range(200))
        out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True)
        rows = [[int(x) for x in line.split()] for line in out.stdout.splitlines()]
        assert len(rows) == 200 and all(r[0] == 0 for r in rows)
        return [r[1:] for r in rows]
    return run


@pytest.mark.parametrize("noise, drift", [(0.0, 0.0), (0.01, 0.0), (0.03, 0.0), (0.1, 0.0),
                                          (0.03, 0.001)])
def test_equal_variants_stay_untuned(plans, noise, drift):
    """At most one search in a hundred may come back with a plan by chance."""
    tuned = sum(any(p) for p in plans(noise, drift, -1, 0.0))
    assert tuned <= 2, tuned


@pytest.mark.parametrize("cls", [0, 1, 2, 3])
def test_faster_tile_is_found(plans, cls):
    """A tile that saves 5% is found behind 1% of noise, for its class alone."""
    for p in plans(0.01, 0.0, cls, 0.05):
        assert p[cls] & 15 == 1 and all(p[q] == 0 for q in range(4) if q != cls), p
