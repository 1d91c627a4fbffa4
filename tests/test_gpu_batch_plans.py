"""Every tile plan of a batch against the single runs, which no plan reaches: bit
for bit the same states and next steps (plan value 0 is a choice for the
instance's share of the chip, vlct_step's one for the whole chip)."""
import numpy as np
import pytest

from oracle import ref
from parity_util import FIELDS
from test_gpu_batch import _instances, _need_gpu, _run_plan, _single

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("recon", [2, 5])
@pytest.mark.parametrize("plan", [0x00, 0x01, 0x02, 0x10, 0x11, 0x12, 0x20, 0x21, 0x22])
def test_plan_equals_single_runs(plan, recon):
    _need_gpu()
    inst = _instances(recon)
    dts = [ref.cfl_dt(g, s) for g, s in inst]
    outs, nexts = _run_plan(inst, dts, [plan] * len(inst), nsteps=2)
    for q, ((g, s), dt) in enumerate(zip(inst, dts)):
        want, single_nexts, _ = _single(g, s, dt, 2)
        assert [float(n[q]) for n in nexts] == single_nexts, q
        for f in FIELDS:
            assert np.array_equal(outs[q][f], want[f]), (q, f)
