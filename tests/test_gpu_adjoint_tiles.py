"""The adjoint where its blocks and segments end: rows one short of, equal to
and one longer than a one-wave block of the x kernels (62 to 65 cells) and a
256-item block (254 to 256), march segments of 1, 5 and 32 cells, taped and
untaped, against the complex step of the oracle along random directions within
the 1e-10 of the other adjoint tests (both sides exact to rounding)."""
import numpy as np
import pytest

from oracle import ref
from paper_2402_05240_amd import inputs as I
from parity_util import FIELDS
from test_gpu_adjoint import _gpu_vjp, _need_gpu, _random_cotangent, cso  # noqa: F401
from test_gpu_parity import _shaped_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, admarch", [
    ((62, 3, 7), 1), ((63, 2, 3), 5), ((64, 5, 2), 32), ((65, 4, 6), 5), ((254, 2, 3), 1),
    ((255, 3, 2), 32), ((256, 2, 2), 5)])
@pytest.mark.parametrize("recon", [1, 2, 3, 4, 5])
def test_adjoint_block_and_segment_edges(cso, recon, shape, admarch, monkeypatch):  # noqa: F811
    _need_gpu()
    import torch
    from paper_2402_05240_amd.autograd import Simulator
    monkeypatch.setenv("VLCT_TILES", "admarch=%d" % admarch)
    g, s = _shaped_state(shape, recon, (0, 0, 0), 31)
    dt = ref.cfl_dt(g, s)
    lam = _random_cotangent(g, 32)
    lin = _gpu_vjp(g, s, lam, dt)
    sim = Simulator(g)
    up = [torch.from_numpy(np.ascontiguousarray(s[f])).cuda() for f in FIELDS]
    lup = [torch.from_numpy(np.ascontiguousarray(lam[f])).cuda() for f in FIELDS]
    dtd, tape = torch.tensor([dt], dtype=torch.float64, device="cuda:0"), sim.new_tape()
    sim.step_taped(up, dtd, tape)
    taped = dict(zip(FIELDS, (t.cpu().numpy() for t in sim.adjoint_taped(up, lup, dtd, tape))))
    rng = np.random.default_rng(33)
    for _ in range(2):
        delta = {f: rng.standard_normal(g.field_shape(f)) for f in FIELDS}
        I._periodic_face_copy(g, delta)
        _, jv, st = cso.jvp(g, s, delta, [dt])
        assert st == 0
        want = sum(float(np.sum(lam[f] * jv[f])) for f in FIELDS)
        scale = sum(float(np.sum(np.abs(lam[f] * jv[f]))) for f in FIELDS)
        for got in (lin, taped):
            err = abs(sum(float(np.sum(got[f] * delta[f])) for f in FIELDS) - want) / scale
            assert err <= 1e-10, (recon, shape, admarch, err)
