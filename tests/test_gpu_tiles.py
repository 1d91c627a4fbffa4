"""The step's tiles and segments at the sizes where they end: sides of one cell,
one below, at and above a tile's 13 rows and 32 columns, a row's 254 cells and
a march's segments; each forced choice (VLCT_TILES) against the automatic one
bit for bit (the tiles only regroup the same arithmetic), and that against the
oracle at the bar of the parity tests (rounding of two steps)."""
import dataclasses

import numpy as np
import pytest

from paper_2402_05240_amd import inputs as I
from parity_util import FIELDS
from test_gpu_parity import _check, _gpu_run, _need_gpu, _oracle_run

pytestmark = pytest.mark.gpu

VARIANTS = ["ct=1,march=1,pred=1", "ct=2,march=2,pred=2,predtile=14,cttile=14",
            "ct=3,march=3,pred=5,predtile=31,cttile=30", "march=13,predtile=126,cttile=126",
            "march=32,predtile=1,cttile=1,ct=7", "pred=4096,ct=4096,predtile=13,cttile=20"]


@pytest.mark.parametrize("n, recon, outflow", [
    ((1, 2, 13), 2, False), ((14, 13, 1), 1, True), ((33, 14, 3), 4, False),
    ((32, 26, 17), 5, True), ((31, 12, 33), 1, False), ((254, 3, 2), 3, False),
    ((255, 4, 2), 2, True), ((12, 27, 35), 3, True)])
def test_tile_edges(n, recon, outflow, monkeypatch):
    _need_gpu()
    g, s0 = I.blast(n, b0=1.0, recon=recon)
    if not outflow:
        g = dataclasses.replace(g, bc=(0, 0, 0))
    orc, dts, _, status = _oracle_run(g, s0, nsteps=2)
    monkeypatch.delenv("VLCT_TILES", raising=False)
    base, nexts, st = _gpu_run(g, s0, dts)
    assert st == status
    _check(g, s0, base, orc)
    for v in VARIANTS:
        print(n, v, flush=True)
        monkeypatch.setenv("VLCT_TILES", v)
        got, nv, stv = _gpu_run(g, s0, dts)
        for f in FIELDS:
            assert np.array_equal(got[f], base[f]), (v, f)
        assert nv == nexts and stv == st, v
