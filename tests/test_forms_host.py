"""Each form of the device physics header that is written otherwise than the
oracle's, against the oracle on random data: the half-slope PLM limiter, PPM
with the common sign factored out of its curvature limiter, HLLD evaluating one
side after the selection; with the library's roots and quotients, and with the
device's own refinement chains.  Both sides round every operation, in different
orders: the bound is the 1e-12 of the other host checks of the header."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import ref
from test_oracle_units import GAM

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_05240_amd", "csrc")
CHAINS = ["VLCT_HOST_COUNT", "VLCT_HOST_ESTIMATES"]


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("forms_probe")
    for c in CHAINS:
        subprocess.run([gxx, "-O1", "-std=c++17", "-ffp-contract=off", "-D" + c, "-I", CSRC, "-o",
                        str(d / c), os.path.join(HERE, "physics_check", "forms_probe.cpp")],
                       check=True)

    def run(chains, form, cases):
        text = "\n".join(" ".join("%.17g" % x for x in np.ravel(c)) for c in cases)
        out = subprocess.run([str(d / chains), form], input=text, check=True,
                             capture_output=True, text=True).stdout
        rows = np.array([[float(x) for x in line.split()] for line in out.splitlines()])
        assert len(rows) == len(cases)
        return rows
    return run


def _states(rng, n, spread):
    """n neighbouring cells about one random state, smooth or with a jump."""
    w = np.array([rng.uniform(0.3, 3.0), *rng.normal(0, 1, 3), rng.uniform(0.1, 3.0),
                  *rng.normal(0, 1, 2)])
    j = np.arange(n) - n // 2
    if rng.uniform() < 0.6:
        d, c = rng.normal(0, spread, 7) * np.abs(w).clip(0.1), rng.normal(0, 1, 3)
        s = w + np.outer(c[0] * j + c[1] * j ** 2 + c[2] * j ** 3 / 4, d)
    else:
        s = w * (1 + rng.normal(0, spread / 3, (n, 7)))
        s[j >= rng.integers(1 - n // 2, n // 2 + 1)] += rng.normal(0, 0.3, 7) * np.abs(w).clip(0.1)
    s[:, 0], s[:, 4] = np.abs(s[:, 0]) + 0.05, np.abs(s[:, 4]) + 0.05
    return s


@pytest.mark.parametrize("form", ["plmc", "plmp", "ppmc", "ppmp"])
@pytest.mark.parametrize("chains", CHAINS)
def test_reconstruction_form(probe, chains, form):
    rng = np.random.default_rng(61)
    sten = [_states(rng, 3 if form[:3] == "plm" else 5, spread)
            for spread in (0.3, 0.05, 1e-4) for _ in range(300)]
    bns = rng.normal(0, 1, len(sten))
    rows = probe(chains, form, [np.append(s.ravel(), [b, GAM]) for s, b in zip(sten, bns)])
    for q, (s, b) in enumerate(zip(sten, bns)):
        args = (s,) if form == "plmp" else (s, b, GAM)
        om, op = getattr(ref, form)(*args)
        tol = 1e-12 * (np.abs(s).max() + 1.0)
        assert np.abs(rows[q, :7] - om).max() <= tol, q
        assert np.abs(rows[q, 7:] - op).max() <= tol, q


@pytest.mark.parametrize("chains", CHAINS)
def test_hlld_form(probe, chains):
    rng = np.random.default_rng(62)
    cases = []
    for q in range(1000):
        l, r = _states(rng, 3, 0.3)[:2]
        shift = rng.uniform(-6, 6) if q % 2 else 0.0   # every fan region
        l[1] += shift
        r[1] += shift
        cases.append(np.concatenate([l, r, [rng.uniform(-2, 2), GAM]]))
    rows = probe(chains, "hlld", cases)
    for c, row in zip(cases, rows):
        f = ref.hlld(c[:7], c[7:14], c[14], c[15], with_upwind=True)
        f, up = f[:7], f[7]
        assert np.abs(row[:7] - f).max() <= 1e-12 * (np.abs(f).max() + 1.0)
        assert row[7] == up


def test_ppm_curvature_limiter(probe):
    """min(C|da|, C|db|, |d2|), C = 1.25, where all three have one sign, else
    zero: exactly, ties, zeros of either sign and far-apart magnitudes included."""
    rng = np.random.default_rng(63)
    vals = [0.0, -0.0, 1.0, -1.0, 1.25, 0.8, 1e-200, -1e-200, 1e200, -1e200, 5e-324]
    cases = [(a, b, c) for a in vals for b in vals for c in vals]
    cases += [tuple(x) for x in rng.normal(0, 1, (3000, 3))]
    rows = probe("VLCT_HOST_COUNT", "curv", cases)[:, 0]
    for (d2, da, db), got in zip(cases, rows):
        one = np.sign(d2) == np.sign(da) == np.sign(db) != 0
        assert got == (min(1.25 * abs(da), 1.25 * abs(db), abs(d2)) if one else 0.0), (d2, da, db)
